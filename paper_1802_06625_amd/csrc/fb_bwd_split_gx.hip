// Input gradient of the filter bank on the half-precision matrix cores with
// split operands (prune_fb_backward), for filters of 15 to 64 taps.
//
// With g = grad_y, r = |x| and powers p of the basis |x|^p x,
//   G_p[m] = sum_l conj(h_p[l]) g[m + l]             (outputs of the frame)
//   P = sum_p r^p G_p,   Q = sum_p (p/2) r^p G_p
//   grad_x[m] = P + Q + (x^2/r^2) conj(Q).
// G_p is the forward's block product run backwards (fb_split.hip): rows are 16
// phases x (re, im), columns blocks of 16 NT samples and the contraction 8 S
// positions x (re, im) on v_mfma_f32_32x32x16_f16; the taps' Toeplitz matrix
// runs forward in time and the Hankel matrix is g's.  g does not depend on the
// power: its two half-precision parts are written to the wave's LDS planes
// once and serve every power; P is a Horner sum over the powers, from the
// highest down, in fp32 registers, and Q = (r/2) dP/dr its derivative's.  Taps
// of several banks are added first (the sum over banks of one power).
//
// Precision.  As in the forward: g scaled by a power of two per wave (and r, so
// that its powers stay below one), the taps per power, high x high + low x high
// + high x low summed per power with the low products first.  Relative error
// against fp64 for 15 to 64 taps: 0.9e-7 to 1.3e-7 for one power, 2.2e-7 to
// 2.5e-7 for eight of constant envelope, where products of fp32 have 1.0e-7 to
// 2.3e-7 and 2.4e-7 to 2.9e-7.  What g's parts can miss of it (2^-25 of the
// scaled g a tap, as in the forward) is compared with the outputs: with HS_p
// the sum of the magnitudes of power p's scaled taps and T = 2^-25 sum_p
// 1.5 (1 + p) HS_p r^p, outputs whose |P| is below 2^17 T are evaluated one by
// one in fp32 instead; a wave that has more than kFew of them, or a lane with
// all of its outputs (sixteen of 32 in a row) below 2^20 T, takes products of
// fp32 on the matrix core, and so does a wave whose g or taps are not finite or
// beyond 2^93, or whose |x| reaches 2^59 or is not zero and below 2^-59.
// Outputs from which on g is zero over the filter's length are exact zeros and
// stay.  Gaussian samples have their |P|'s median near 2^33 T.
//
// What bounds it.  1024 frames x 32768 of 64 streams, 30 % of them skipped, 64
// taps, 7 powers: 394 us, from 790 us for products of fp32 on the matrix core
// (k_bwd_gu_mfma); 256 frames x 8192, 16 taps, 8 powers: 42 us from 56.  The
// matrix core takes 155 us of the former, the LDS 160 us, the vector unit 100
// us, the samples 170 us at the copy rate, and a pass's loads and sums lie
// before and after its products: two waves a SIMD overlap them in part.  Lanes
// reading x and writing gradients in the products' layout, two samples from
// each of 32 columns: 15 us more.  Groups of 8 or 16 tiles a ticket: 6 and 48
// us more (uneven ends).
#include "bwd_common.h"
#include "runtime_kernels.h"
#include "split_common.h"

namespace prune {

namespace {
constexpr int kGxWaves = 4;
constexpr int kGxPow = 10;                       // powers of a bank
constexpr int kGxTab = PRUNE_MAX_L + 32;         // table entries per power: 8 S + 16 at most
constexpr int kGxGroup = kGxWaves;               // list entries per ticket
constexpr int kTapBits = 15, kCotBits = 15;      // largest tap and cotangent component scaled below 2^15
constexpr float kGxMargin = 0x1p-8f;             // 2^17 times an operand's 2^-25
constexpr float kHuge = 3e38f;
constexpr int kNoTap = -100000, kBadTap = 100000;
constexpr uint32_t kTinyX = 8u << 23, kLargeX = (127u + 119u) << 23;   // |x|^2 from 2^-119 to 2^119 (or zero)

struct GxShared {
  uint32_t tab[kGxPow][2][2][kGxTab];            // [power][high, low part][re, im row][tap + 15]
  int cexp[16];                                  // per power: its largest tap is below 2^cexp
  int hsum[16];                                  // per power: HS_p, and 2^16 for each component below one half
  BwdFrame frame[2][kGxGroup];                   // the entries of this group and of the next
  int n0[2][kGxGroup];
  uint32_t at[2][kGxGroup];                      // frame index
  uint32_t next[2];
};

// LDS word of window sample 2 lane + 128 i: one pad chunk of four samples per
// column of 16 NT samples.
template <int NT>
__device__ __forceinline__ int gx_idx(int lane, int i) {
  return 2 * lane + 4 * (2 * lane / (16 * NT)) + (128 + 4 * (8 / NT)) * i;
}
constexpr int gx_plane(int nt) { return (4 * nt + 1) * (128 + 4 * (8 / nt)); }

// Conjugate taps of a frame: every power of its bank when a single bank is
// active, the sums over the banks of its mask's branches otherwise.
__device__ __forceinline__ void gx_table(const prune_fb_desc &d, const BwdFrame &F, uint32_t Lmax, int bank1, int S,
                                         GxShared &sh) {
  const int TS = 8 * S + 16;
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  if (t < 16) {
    sh.cexp[t] = kNoTap;
    sh.hsum[t] = 0;
  }
  __syncthreads();
  float2 h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = t + 64 * kGxWaves * i, p = k / TS, l = k - p * TS - 15;
    h[i] = make_float2(0.f, 0.f);
    if (p < (int)d.Kmax && l >= 0) {
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        const bool on = bank1 >= 0 ? (int)bank == bank1 : ((F.mask >> (bank * d.Kmax + p)) & 1u) != 0;
        if (on && l < (int)d.L[bank]) {
          const float2 z = ld_global(F.taps + (size_t)(bank * d.Kmax + p) * Lmax + l);
          h[i].x += z.x;
          h[i].y += z.y;
        }
      }
      const uint32_t hb = max(abs_bits(h[i].x), abs_bits(h[i].y));
      if (hb >= kHigh) atomicMax(&sh.cexp[p], kBadTap);
      else if (hb) atomicMax(&sh.cexp[p], (int)(hb >> 23) - 126);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = t + 64 * kGxWaves * i, p = k / TS, q = k - p * TS;
    if (p < kGxPow) {
      const int sc = kTapBits - sh.cexp[p];
      const float hr = ldexpf(h[i].x, sc), hi = ldexpf(h[i].y, sc), ar = fabsf(hr), ai = fabsf(hi);
      if (ar + ai > 0.f && sh.cexp[p] != kBadTap)
        atomicAdd(&sh.hsum[p], (int)ceilf(ar + ai) + (ar > 0.f && ar < 0.5f ? 1 << 16 : 0) +
                                   (ai > 0.f && ai < 0.5f ? 1 << 16 : 0));
      const _Float16 r1 = (_Float16)hr, i1 = (_Float16)hi;
      const _Float16 r2 = (_Float16)(hr - (float)r1), i2 = (_Float16)(hi - (float)i1);
      sh.tab[p][0][0][q] = __builtin_bit_cast(uint32_t, half2v{r1, i1});
      sh.tab[p][0][1][q] = __builtin_bit_cast(uint32_t, half2v{(_Float16)-i1, r1});
      sh.tab[p][1][0][q] = __builtin_bit_cast(uint32_t, half2v{r2, i2});
      sh.tab[p][1][1][q] = __builtin_bit_cast(uint32_t, half2v{(_Float16)-i2, r2});
    }
  }
  __syncthreads();
}

// A frame's entry in scalar registers.
__device__ __forceinline__ BwdFrame uniform_frame(const BwdFrame &f) {
  auto u32 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  auto ptr = [&](const float2 *p) {
    const uint64_t v = (uint64_t)p;
    return (float2 *)((uint64_t)u32((uint32_t)(v >> 32)) << 32 | u32((uint32_t)v));
  };
  BwdFrame r;
  r.x = ptr(f.x); r.g = ptr(f.g); r.gx = ptr(f.gx); r.taps = ptr(f.taps);
  r.n = u32(f.n); r.mask = u32(f.mask); r.route = u32(f.route); r.t0 = u32(f.t0);
  r.stream = r.pad0 = r.pad1 = r.pad2 = 0;
  return r;
}

// Where a pass's gradients go: grad_x at positions [0, n), or the halo row
// (positions [-H, 0)).
struct GxOut {
  float2 *gx;       // position 0
  int lo, hi;       // positions written
};

// FAST: |x|^2 is zero or within [1e-36, 1e36].
template <bool FAST>
__device__ __forceinline__ float2 gx_combine(float xr, float xi, float pr, float pi, float qr, float qi) {
  const float r2 = xr * xr + xi * xi, nr = xr * xr - xi * xi, ni = 2.f * xr * xi;
  float er = 0.f, ei = 0.f;   // x^2 / r^2
  if constexpr (FAST) {
    const float y = __builtin_amdgcn_rcpf(fmaxf(r2, 1e-36f));
    er = nr * y;
    ei = ni * y;
    er = fmaf(fmaf(-r2, er, nr), y, er);   // the quotients to half a unit in the last place or so
    ei = fmaf(fmaf(-r2, ei, ni), y, ei);
  } else if (r2 > 0.f) {
    er = nr / r2;
    ei = ni / r2;
  }
  return make_float2(pr + qr + (er * qr + ei * qi), pi + qi + (ei * qr - er * qi));
}

// Up to kBT samples, of g or zeros, by one wave: every load before the stores.
__device__ __forceinline__ void copy_out(const float2 *g, GxOut o, int lane) {
  pair_u v[kBT / 128];
#pragma unroll
  for (int i = 0; i < kBT / 128; ++i) {
    const int m = o.lo + 128 * i + 2 * lane;
    v[i] = pair_u{0.f, 0.f, 0.f, 0.f};
    if (g && m + 1 < o.hi) v[i] = ld_pair(g + m);
    else if (g && m < o.hi) v[i].x = ld_global(g + m).x, v[i].y = ld_global(g + m).y;
  }
#pragma unroll
  for (int i = 0; i < kBT / 128; ++i) {
    const int m = o.lo + 128 * i + 2 * lane;
    if (m + 1 < o.hi) st_pair(o.gx + m, v[i]);
    else if (m < o.hi) st_global(o.gx + m, make_float2(v[i].x, v[i].y));
  }
}

// A wave's gradients at positions wb .. wb + 512 nt - 1 from products of fp32
// (16 x 16 blocks, steps of four positions, three real products a complex one).
// g has a pad word per 16 in the planes (a step's lanes read 16 words apart);
// a branch's taps, zeros on either side, follow it.
constexpr int kGxTapAt = (512 * 2 + 80) / 16 * 17, kGxTapLen = PRUNE_MAX_L + 32;
__device__ __noinline__ void gx_fp32(const prune_fb_desc &d, const BwdFrame &F, uint32_t Lmax, int wb, int nt, GxOut o,
                                     float *plane, int pitch, int lane) {
  const int n = (int)F.n, li = lane & 15, lk = lane >> 4;
  const uint32_t kfull = (1u << d.Kmax) - 1u;
  wave_lds_fence();
  for (int k = lane; k < 512 * nt + 80; k += 64) {
    const int q = wb + k;
    const float2 v = q >= 0 && q < n ? ld_global(F.g + q) : make_float2(0.f, 0.f);
    plane[k + (k >> 4)] = v.x;
    plane[pitch + k + (k >> 4)] = v.y;
  }
  wave_lds_fence();
  for (int t = 0; t < 2 * nt; t += 2) {   // two blocks of 256 at a time
    const int m0 = wb + 256 * t + 16 * li + 4 * lk;
    float xr[2][4], xi[2][4], rr[2][4], pr[2][4], pi[2][4], qr[2][4], qi[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 256 * u + e;
        const float2 v = m < n && m >= -(int)F.t0 ? ld_global(F.x + m) : make_float2(0.f, 0.f);
        xr[u][e] = v.x;
        xi[u][e] = v.y;
        rr[u][e] = sqrtf(v.x * v.x + v.y * v.y);
        pr[u][e] = pi[u][e] = qr[u][e] = qi[u][e] = 0.f;
      }
    for (int p = (int)d.Kmax - 1; p >= 0; --p) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          pr[u][e] *= rr[u][e];
          pi[u][e] *= rr[u][e];
          qr[u][e] *= rr[u][e];
          qi[u][e] *= rr[u][e];
        }
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        if (!((F.mask >> (bank * d.Kmax)) & kfull & (1u << p))) continue;
        const int L = (int)d.L[bank];
        const float2 *tb = F.taps + (size_t)(bank * d.Kmax + p) * Lmax;
        wave_lds_fence();
        for (int k = lane; k < kGxTapLen; k += 64) {
          const float2 h = k >= 16 && k - 16 < L ? ld_global(tb + (k - 16)) : make_float2(0.f, 0.f);
          plane[kGxTapAt + k] = h.x;
          plane[pitch + kGxTapAt + k] = h.y;
        }
        wave_lds_fence();
        floatx4 a0[2], a1[2], a2[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) a0[u] = a1[u] = a2[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < (L + 15 + 3) / 4; ++s) {
          const int l = kGxTapAt + 16 + 4 * s + lk - li;
          const float hr = plane[l], hi = plane[pitch + l];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int k = 256 * (t + u) + 16 * li + 4 * s + lk, w = k + (k >> 4);
            const float gr = plane[w], gi = plane[pitch + w];
            a0[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(hr, gr, a0[u], 0, 0, 0);
            a1[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(-hi, gi, a1[u], 0, 0, 0);
            a2[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(hr - hi, gr + gi, a2[u], 0, 0, 0);
          }
        }
        const float ph = 0.5f * (float)p;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gr = a0[u][e] - a1[u][e], gi = a2[u][e] - a0[u][e] - a1[u][e];
            pr[u][e] += gr;
            pi[u][e] += gi;
            qr[u][e] = fmaf(ph, gr, qr[u][e]);
            qi[u][e] = fmaf(ph, gi, qi[u][e]);
          }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 256 * u + e;
        if (m >= o.lo && m < o.hi)
          st_global(o.gx + m, gx_combine<false>(xr[u][e], xi[u][e], pr[u][e], pi[u][e], qr[u][e], qi[u][e]));
      }
  }
  wave_lds_fence();
}

// A lane's output b of a wave (in the order of gx_pass): its place from wb.
template <int NT>
__device__ __forceinline__ int output_at(int lane, int b) {
  return 16 * NT * (lane & 31) + 2 * (lane >> 5) + 16 * (b >> 3) + 4 * ((b >> 1) & 3) + (b & 1);
}

// The outputs in `few` (a bit for each of the lane's) by the definition in fp32,
// one after another, a lane for each tap.
template <int NT>
__device__ __noinline__ void fix_outputs(const prune_fb_desc &d, const BwdFrame &F, uint32_t Lmax, int wb, GxOut o,
                                         uint32_t few, int lane) {
  const int n = (int)F.n;
  for (;;) {
    const unsigned long long who = __ballot(few != 0u);
    if (!who) break;
    const int src = __ffsll(who) - 1, b = __ffs(__builtin_amdgcn_readlane((int)few, src)) - 1;
    const int m = wb + output_at<NT>(src, b), q = m + lane;
    const float2 x = m >= -(int)F.t0 ? ld_global(F.x + m) : make_float2(0.f, 0.f);   // (m < n)
    const float2 g = q >= 0 && q < n ? ld_global(F.g + q) : make_float2(0.f, 0.f);
    const float r = sqrtf(x.x * x.x + x.y * x.y);
    float pr = 0.f, pi = 0.f, qr = 0.f, qi = 0.f;
    for (int p = (int)d.Kmax - 1; p >= 0; --p) {
      float gr = 0.f, gi = 0.f;
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        const uint32_t br = bank * d.Kmax + p;
        if (!((F.mask >> br) & 1u) || lane >= (int)d.L[bank]) continue;
        const float2 h = ld_global(F.taps + (size_t)br * Lmax + lane);
        gr += fmaf(h.x, g.x, h.y * g.y);
        gi += fmaf(h.x, g.y, -h.y * g.x);
      }
      for (int k = 32; k; k >>= 1) {
        gr += __shfl_xor(gr, k, 64);
        gi += __shfl_xor(gi, k, 64);
      }
      const float ph = 0.5f * (float)p;
      pr = fmaf(pr, r, gr);
      pi = fmaf(pi, r, gi);
      qr = fmaf(qr, r, ph * gr);
      qi = fmaf(qi, r, ph * gi);
    }
    if (lane == 0) st_global(o.gx + m, gx_combine<false>(x.x, x.y, pr, pi, qr, qi));
    if (lane == src) few &= few - 1u;
  }
}

// Whether g is zero over the L samples from each output in `zeros` (a bit for
// each of the lane's) on.
template <int NT>
__device__ __noinline__ bool silent_after(const BwdFrame &F, int wb, int L, uint32_t zeros, uint32_t *plane, int lane) {
  const int n = (int)F.n;
  const unsigned long long ge = ~0ull << lane, gt = lane < 63 ? ~0ull << (lane + 1) : 0ull;
  auto low = [](unsigned long long m) { return m ? __ffsll(m) - 1 : 1 << 20; };
  int next = 1 << 20;                          // the first sample after this run that is not zero
  wave_lds_fence();
  for (int i = 4 * NT; i >= 0; --i) {
    unsigned long long on[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int p = wb + 2 * lane + 128 * i + q;
      const float2 z = p >= 0 && p < n ? ld_global(F.g + p) : make_float2(0.f, 0.f);
      on[q] = __ballot((abs_bits(z.x) | abs_bits(z.y)) != 0u);
    }
    const int k = 128 * i, odd = 2 * low(on[1] & ge) + 1;
    plane[k + 2 * lane] = (uint32_t)min(next, k + min(odd, 2 * low(on[0] & ge)));
    plane[k + 2 * lane + 1] = (uint32_t)min(next, k + min(odd, 2 * low(on[0] & gt)));
    next = min(next, k + min(2 * low(on[0]), 2 * low(on[1]) + 1));
  }
  wave_lds_fence();
  bool ok = true;
  for (int b = 0; b < 8 * NT; ++b) {
    const int k = output_at<NT>(lane, b);
    if ((zeros >> b) & 1u) ok &= (int)plane[k] - k >= L;
  }
  wave_lds_fence();
  return !__any(!ok);
}

// One pass of one wave: positions wb .. wb + 512 NT - 1 (32 columns of 16 NT).
// kPassLeft: nothing is written, the outputs are left to gx_fp32.  kPassCheck:
// everything is written; the outputs in the upper half of `flags` (a bit for
// each of the lane's) are to be evaluated again, and where g is not zero after
// one in the lower half (silent_after), all are left to gx_fp32.
enum { kPassDone, kPassLeft, kPassCheck };
constexpr int kFew = 12;
template <int NT, int S, int PLANE>
__device__ __forceinline__ int gx_pass(const BwdFrame &F, int wb, uint32_t pm, GxOut o, const GxShared &sh,
                                       uint32_t *__restrict__ plane, int lane, uint32_t &flags) {
  constexpr int NP = 4 * NT + 1;               // sample pairs per lane
  constexpr int NC = 2 * NT + S - 2;           // chunk pairs per column
  constexpr int CW = 4 * NT;                   // chunks per column
  asm volatile("" : "+v"(lane));
  const int n = (int)F.n, li = lane & 31, g = lane >> 5;
  pair_u v[NP];
  if (wb >= 0 && wb + 512 * NT + 128 <= n) {
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = ld_pair(F.g + wb + 2 * lane + 128 * i);
  } else {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      float2 z[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int p = wb + 2 * lane + 128 * i + q;
        z[q] = p >= 0 && p < n ? ld_global(F.g + p) : make_float2(0.f, 0.f);
      }
      v[i] = pair_u{z[0].x, z[0].y, z[1].x, z[1].y};
    }
  }
  // Sample pairs of x, P and Q change places through the LDS: lane l's pair k
  // is pair l & 7 of column 8 (k & 3) + (l >> 3) in result tile k >> 2, whole
  // cache lines of memory.  One pad pair per column and tile.
  const bool inside = wb >= -(int)F.t0 && wb + 512 * NT <= n;
  const int cp = wb + 16 * NT * (lane >> 3) + 2 * (lane & 7);
  auto pair_at = [&](int k) { return cp + 128 * NT * (k & 3) + 16 * (k >> 2); };
  auto load_x = [&](int k) -> pair_u {
    const int m = pair_at(k);
    if (inside) return ld_pair(F.x + m);
    const float2 a = m < n && m >= -(int)F.t0 ? ld_global(F.x + m) : make_float2(0.f, 0.f);
    const float2 b = m + 1 < n && m + 1 >= -(int)F.t0 ? ld_global(F.x + m + 1) : make_float2(0.f, 0.f);
    return pair_u{a.x, a.y, b.x, b.y};
  };
  const int mine = 9 * li + g;                 // this lane's pair 0 in the products' layout; pair q at + 2 q
  const int turn = 9 * (lane >> 3) + (lane & 7);   // in the memory's: pair k of a tile at + 72 k
  float rr[NT][8];
  uint32_t s_min = ~0u, s_max = 0;             // |x|^2 as bits; a zero passes as the largest of the minima
  {
    pair_u x[4 * NT];
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) x[k] = load_x(k);
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) {
      floatx2 r;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float re = q ? x[k].z : x[k].x, im = q ? x[k].w : x[k].y, s2 = fmaf(re, re, im * im);
        const uint32_t b = __builtin_bit_cast(uint32_t, s2);
        s_min = min(s_min, b - 1u);
        s_max = max(s_max, b);
        const float y = __builtin_amdgcn_rsqf(fmaxf(s2, 1e-37f)), r0 = s2 * y;
        r[q] = fmaf(fmaf(-r0, r0, s2), 0.5f * y, r0);
      }
      *(floatx2 *)(plane + 2 * (288 * (k >> 2) + turn + 72 * (k & 3))) = r;
    }
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const floatx2 z = *(const floatx2 *)(plane + 2 * (288 * j + mine + 2 * q));
        rr[j][2 * q] = z.x;
        rr[j][2 * q + 1] = z.y;
      }
  }
  const uint32_t S2 = (uint32_t)wave_max((int)min(s_max, kInf));   // the largest |x|^2, or not finite
  const int ex = S2 ? ((int)(S2 >> 23) - 125) >> 1 : 0;            // |x| < 2^ex
  const float rs = ldexpf(1.f, -ex);
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 8; ++q) rr[j][q] *= rs;
  uint32_t am = 0;
#pragma unroll
  for (int i = 0; i < NP; ++i)
    am = max(max(am, max(abs_bits(v[i].x), abs_bits(v[i].y))), max(abs_bits(v[i].z), abs_bits(v[i].w)));
  const uint32_t A = (uint32_t)wave_max((int)am);
  const int e = A >= kLow ? (int)(A >> 23) - 126 : 0;   // |re|, |im| < 2^e
  int ep = kNoTap;
  if (lane < kGxPow && ((pm >> lane) & 1u)) ep = sh.cexp[lane];
  if (__any(ep == kBadTap) || (A != 0 && (A < kLow || A >= kHigh)) || S2 >= kLargeX || __any(s_min < kTinyX))
    return kPassLeft;
  ep += lane * ex;
  const int eb = wave_max(ep);
  const float ef = ldexpf(1.f, max(ep - eb, -200));
  float neg1 = -1.f;
  asm volatile("" : "+v"(neg1));
  const float gs = __builtin_bit_cast(float, (uint32_t)(127 + kCotBits - e) << 23);
  wave_lds_fence();
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    uint32_t hi[2], lo[2];
    split_pair(v[i] * gs, neg1, hi, lo);
    const int q = gx_idx<NT>(lane, i);
    *(uintx2 *)(plane + q) = uintx2{hi[0], hi[1]};
    *(uintx2 *)(plane + PLANE + q) = uintx2{lo[0], lo[1]};
  }
  wave_lds_fence();
  const uint32_t *trow = &sh.tab[0][0][li & 1][15 - (li >> 1) + 4 * g];
  const uint32_t *brow = plane + (CW + 1) * 4 * li + 4 * g;
  float P[NT][16], Q[NT][16];                  // sum of r^p G_p and its derivative by r
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) P[j][q] = Q[j][q] = 0.f;
  // (written out: the compiler takes a multiply-add that overwrites its addend,
  // and copies P first)
  auto derive = [&]() {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q)
        asm("v_fma_f32 %0, %0, %1, %2" : "+v"(Q[j][q]) : "v"(rr[j][q >> 1]), "v"(P[j][q]));
  };
  auto skip = [&]() {                          // a power without a branch
    derive();
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) P[j][q] *= rr[j][q >> 1];
  };
  int p = 31 - __clz(pm);
  for (uint32_t rest = pm;;) {
    derive();
    const uint32_t *tp = trow + p * (4 * kGxTab);
    floatx16 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
    half8 ah[S], al[S], bh[NC], bl[NC];
    auto fetch = [&](int odd) {
#pragma unroll
      for (int s = odd; s < S; s += 2) {
        ah[s] = __builtin_bit_cast(half8, *(const uintx4_u *)(tp + 8 * s));
        al[s] = __builtin_bit_cast(half8, *(const uintx4_u *)(tp + 2 * kGxTab + 8 * s));
      }
#pragma unroll
      for (int i = odd; i < NC; i += 2) {
        const int w = 4 * (2 * i + 2 * i / CW);
        bh[i] = __builtin_bit_cast(half8, *(const uintx4 *)(brow + w));
        bl[i] = __builtin_bit_cast(half8, *(const uintx4 *)(brow + PLANE + w));
      }
    };
    auto mma = [&](int odd, const half8 *a, const half8 *b) {
#pragma unroll
      for (int i = odd; i < NC; i += 2)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (i - 2 * j >= 0 && i - 2 * j < S)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i - 2 * j], b[i], acc[j], 0, 0, 0);
    };
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
      fetch(odd);
      mma(odd, al, bh);
      mma(odd, ah, bl);
      mma(odd, ah, bh);
    }
    const float f = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ef), p));
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) P[j][q] = fmaf(P[j][q], rr[j][q >> 1], acc[j][q] * f);   // f: a power of two
    rest &= ~(1u << p);
    const int next = rest ? 31 - __clz(rest) : -1;
    for (int k = p - 1; k > next; --k) skip();
    if (next < 0) break;
    p = next;
  }
  // the outputs against what may be missing of them: against T at the largest
  // r first, and each against its own where that does not settle it (at least
  // 2^-80, so that no power that is missing for its ef or by underflow counts)
  flags = 0;
  if (A != 0 && eb > kNoTap / 2) {
    auto size = [&](int b) {
      const int j = b >> 3, q = 2 * (b & 7), m = wb + output_at<NT>(lane, b);
      return m >= o.lo && m < o.hi ? fmaxf(fabsf(P[j][q]), fabsf(P[j][q + 1])) : kHuge;
    };
    const float tv = (pm >> (lane & 15)) & 1u ? kGxMargin * 1.5f * (1 + (lane & 15)) * ef * (float)sh.hsum[lane & 15] : 0.f;
    auto term = [&](int p) {
      return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tv), p));
    };
    const int top = 31 - __clz(pm);
    const float rm = rs * __builtin_amdgcn_sqrtf(__builtin_bit_cast(float, S2));
    float tm = 0x1p-80f, least = kHuge;
    for (int p = top; p >= 0; --p) tm = fmaf(tm, rm, term(p));
    const bool whole = wb >= o.lo && wb + 512 * NT <= o.hi;   // uniform
#pragma unroll
    for (int b = 0; b < 8 * NT; ++b)
      least = fminf(least, whole ? fmaxf(fabsf(P[b >> 3][2 * (b & 7)]), fabsf(P[b >> 3][2 * (b & 7) + 1])) : size(b));
    if (__any(least < 8.f * fmaxf(tm, 0x1p-80f))) {
      bool quiet = true, some = false;
      int few = 0;
      for (int j = 0; j < NT; ++j) {
        float T[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) T[b] = 0.f;
        for (int p = top; p >= 0; --p) {
          const float t = term(p);
#pragma unroll
          for (int b = 0; b < 8; ++b) T[b] = fmaf(T[b], NT > 1 && j ? rr[NT - 1][b] : rr[0][b], t);
        }
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const float r = NT > 1 && j ? rr[NT - 1][b] : rr[0][b];
          const float m = NT > 1 && j ? size(8 * (NT - 1) + b) : size(b);
          const float thr = r > 0.f || (pm & 1u) ? fmaxf(T[b], 0x1p-80f) : 0.f;
          const bool low = m > 0.f && m < thr;
          few += __popcll(__ballot(low));
          quiet &= m < 8.f * thr || m == kHuge;
          some |= m > 0.f && m < kHuge;
          flags |= low ? 0x10000u << (8 * j + b) : m == 0.f && thr > 0.f ? 1u << (8 * j + b) : 0u;
        }
      }
      if (few > kFew || __any(quiet && some)) return kPassLeft;
    }
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) Q[j][q] *= 0.5f * rr[j][q >> 1];
  const int ys = eb + e - kTapBits - kCotBits;
  const bool full = wb >= o.lo && wb + 512 * NT <= o.hi;   // uniform
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    pair_u x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = load_x(4 * j + k);
    wave_lds_fence();
    floatx4 *const sp = (floatx4 *)plane, *const sq = sp + 288;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sp[mine + 2 * q] = floatx4{P[j][4 * q], P[j][4 * q + 1], P[j][4 * q + 2], P[j][4 * q + 3]};
      sq[mine + 2 * q] = floatx4{Q[j][4 * q], Q[j][4 * q + 1], Q[j][4 * q + 2], Q[j][4 * q + 3]};
    }
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int m = pair_at(4 * j + k);
      const floatx4 p = sp[turn + 72 * k], q = sq[turn + 72 * k];
      const float2 a = gx_combine<true>(x[k].x, x[k].y, p.x, p.y, q.x, q.y);
      const float2 b = gx_combine<true>(x[k].z, x[k].w, p.z, p.w, q.z, q.w);
      const pair_u z = {ldexpf(a.x, ys), ldexpf(a.y, ys), ldexpf(b.x, ys), ldexpf(b.y, ys)};
      if (full || (m >= o.lo && m + 1 < o.hi)) st_pair(o.gx + m, z);
      else if (m >= o.lo && m < o.hi) st_global(o.gx + m, make_float2(z.x, z.y));
      else if (m + 1 >= o.lo && m + 1 < o.hi) st_global(o.gx + m + 1, make_float2(z.z, z.w));
    }
  }
  return __any(flags != 0u) ? kPassCheck : kPassDone;
}
}  // namespace

// List entries 0 .. n_items-1 are the tiles (one wave each); n_items ..
// n_items+n_frames-1 the halo rows: the gradient of the H = Lmax-1 stream
// samples before frame f from f's own outputs, into hg[f][0 .. H) for the
// fix-up kernel.  A ticket is kGxGroup entries; the workgroup's waves share
// those in a row that have one tap table.
__global__ __launch_bounds__(64 * kGxWaves, 2) void k_bwd_gx_split(prune_fb_desc d, const BwdFrame *__restrict__ bf,
                                                                   const WorkItem *__restrict__ items,
                                                                   const uint32_t *__restrict__ n_items,
                                                                   unsigned int *__restrict__ ticket,
                                                                   float2 *__restrict__ hg,
                                                                   const uint32_t *__restrict__ sfirst,
                                                                   float2 *__restrict__ gxs) {
  constexpr int PL = gx_plane(2);
  static_assert(PL >= kGxTapAt + kGxTapLen, "g and a branch's taps fit in a plane");
  static_assert(2 * PL >= 2 * 4 * 288 && gx_plane(1) <= PL, "P and Q of a tile, and one-tile passes, fit in the planes");
  __shared__ GxShared sh;
  __shared__ __align__(16) uint32_t s_plane[kGxWaves][2][PL];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t *plane = s_plane[w][0];
  uint32_t Lmax = 1;
  for (uint32_t b = 0; b < d.n_banks; ++b) Lmax = max(Lmax, d.L[b]);
  const int H = (int)Lmax - 1;
  const uint32_t ni = *n_items, total = ni + (H > 0 ? d.n_frames : 0u), ng = (total + kGxGroup - 1) / kGxGroup;
  const uint32_t kfull = (1u << d.Kmax) - 1u;
  // what the tap table holds: a bank's powers (tab_bank), or the sums of a
  // mask over several banks (tab_bank -1; every bit of the mask may be a branch)
  const float2 *tab_taps = nullptr;
  int tab_bank = -1;
  uint32_t tab_mask = 0, par = 0;
  const bool tickets = 2ull * gridDim.x < ng;
  // a group's entries, read a group ahead
  auto entries = [&](uint32_t grp, uint32_t buf) {
    const uint32_t i = grp * kGxGroup + t;
    if (t >= kGxGroup || i >= total) return;
    const uint32_t frame = i >= ni ? i - ni : items[i].frame;
    sh.n0[buf][t] = i >= ni ? -PRUNE_MAX_L : (int)items[i].tile * kBT;
    sh.at[buf][t] = frame;
    sh.frame[buf][t] = bf[frame];
  };
  uint32_t grp = blockIdx.x, grp1 = blockIdx.x + gridDim.x;
  entries(grp, 0);
  for (; grp < ng; par ^= 1u) {
    __syncthreads();
    if (t == 0) sh.next[par] = tickets ? 2u * gridDim.x + atomicAdd(ticket, 1u) : ng;
    entries(grp1, par ^ 1u);
    const uint32_t n_ent = min(total, (grp + 1) * kGxGroup) - grp * kGxGroup;
    uint32_t mine = 0;   // entries of this group that a wave has taken
    for (uint32_t k = 0; k < n_ent; ++k) {
      const bool halo = grp * kGxGroup + k >= ni;
      const uint32_t frame = sh.at[par][k];
      const BwdFrame F = uniform_frame(sh.frame[par][k]);
      const int n = (int)F.n, n0 = __builtin_amdgcn_readfirstlane(sh.n0[par][k]);
      uint32_t pm = 0;
      int L = 1, nb = 0, bank1 = -1;
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        const uint32_t bm = F.route ? 0u : (F.mask >> (bank * d.Kmax)) & kfull;
        pm |= bm;
        if (bm) { L = max(L, (int)d.L[bank]); ++nb; bank1 = (int)bank; }
      }
      if (nb > 1) bank1 = -1;
      if (halo && (F.route || n == 0)) continue;   // the fix-up skips these frames
      GxOut o;
      o.gx = halo ? hg + (size_t)frame * H + H : F.gx;
      o.lo = halo ? -H : n0;
      o.hi = halo ? 0 : min(n, n0 + kBT);
      const bool my = (mine++ & (kGxWaves - 1)) == (uint32_t)w;
      if (!pm) {   // copied frames and empty masks
        if (my) copy_out(F.route ? F.g : nullptr, o, lane);
        continue;
      }
      const uint32_t tm = bank1 >= 0 ? 0u : F.mask;
      if (F.taps != tab_taps || bank1 != tab_bank || tm != tab_mask) {   // uniform across the workgroup
        tab_taps = F.taps;
        tab_bank = bank1;
        tab_mask = tm;
        __syncthreads();
        gx_table(d, F, Lmax, bank1, L <= 33 ? 6 : L <= 49 ? 8 : 10, sh);
      }
      if (!my) continue;
      const int nt = !halo && n - n0 > 512 ? 2 : 1;
      int end;
      uint32_t flags = 0;
      if (nt == 2) {
        if (L <= 33) end = gx_pass<2, 6, PL>(F, n0, pm, o, sh, plane, lane, flags);
        else if (L <= 49) end = gx_pass<2, 8, PL>(F, n0, pm, o, sh, plane, lane, flags);
        else end = gx_pass<2, 10, PL>(F, n0, pm, o, sh, plane, lane, flags);
      } else {
        if (L <= 33) end = gx_pass<1, 6, PL>(F, n0, pm, o, sh, plane, lane, flags);
        else if (L <= 49) end = gx_pass<1, 8, PL>(F, n0, pm, o, sh, plane, lane, flags);
        else end = gx_pass<1, 10, PL>(F, n0, pm, o, sh, plane, lane, flags);
      }
      if (end == kPassCheck) {
        __builtin_amdgcn_s_waitcnt(0);         // for the outputs that are written again
        asm volatile("" ::: "memory");
        const BwdFrame &f = sh.frame[par][k];
        const uint32_t zeros = flags & 0xffffu;
        if (__any(zeros != 0u) && !(nt == 2 ? silent_after<2>(f, n0, L, zeros, plane, lane)
                                            : silent_after<1>(f, n0, L, zeros, plane, lane)))
          end = kPassLeft;
        else if (nt == 2) fix_outputs<2>(d, f, Lmax, n0, o, flags >> 16, lane);
        else fix_outputs<1>(d, f, Lmax, n0, o, flags >> 16, lane);
      }
      if (end == kPassLeft) gx_fp32(d, sh.frame[par][k], Lmax, n0, nt, o, (float *)plane, PL, lane);
    }
    __syncthreads();
    grp = grp1;
    grp1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.next[par]);
  }
  if (sfirst) bwd_zero_gaps(d, bf, sfirst, gxs);
}

void launch_bwd_gx_split(const prune_fb_desc &d, const BwdFrame *bf, const WorkItem *items,
                         const uint32_t *n_items, unsigned int *ticket, float2 *hg, uint32_t grid,
                         const uint32_t *sfirst, float2 *gx, hipStream_t s) {
  hipLaunchKernelGGL(k_bwd_gx_split, dim3(grid), dim3(64 * kGxWaves), 0, s, d, bf, items, n_items, ticket, hg,
                     sfirst, gx);
}

}  // namespace prune
