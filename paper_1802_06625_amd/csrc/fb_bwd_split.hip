// Tap gradients of the filter bank on the half-precision matrix cores with
// split operands (prune_fb_backward).
//
// With g = grad_y and u_p = |x|^p x, over every output n + l of a frame,
//   grad_h_p[l] = sum_n g[n + l] conj(u_p[n]).
// Rows are taps, columns (power, re / im) and the contraction runs over the
// input positions n, on v_mfma_f32_16x16x32_f16: sixteen positions x (re, im)
// a step, sixteen taps a row tile, eight powers a column group.  The row
// operand is a Hankel matrix of g: four consecutive words of g's plane from
// position n + l on, and row tile t of step s is row tile 0 of step s + t, so
// that a step reads one new operand whatever the number of row tiles.  A
// column holds u_p's words as they are for the real part and rotated, one
// sign changed, for the imaginary part.  The sum does not depend on the bank:
// every bank whose mask holds the power takes its taps from the same result.
//
// Precision.  g and every power of x of a chunk of 256 positions are scaled by
// powers of two so that the largest lies near 2^15, and are the sum of two
// half-precision parts (split_pair).  high x high is summed apart from low x
// high + high x low, exactly but for one rounding per eight terms; a chunk's
// sums are added up in fp32, and the tile partials in fp64 (bwd_common.h).
// Relative error against fp64 for 4 to 64 taps and 2 to 10 powers: 1.5e-7 to
// 2.1e-7, where products of fp32 on the matrix cores had 1.9e-7 to 3.1e-7.
// The parts can miss 2^-25 of a scaled value, so a sum of a chunk misses no
// more than T = 2^-25 of the sum of g's magnitudes (and 2^16 for each component
// of g below one half; its rms is a twentieth of that or less).  Where a run's
// sum of any active power and tap lies below 2^17 of its chunks' T, the run is
// summed by the fp32 definition instead; so is a chunk where x or g is not
// finite or beyond 2^93.  (The check is on a run's sums, not a chunk's: beside a
// masked stretch of g a chunk has sums of a few terms, whatever they are, at
// most filter lengths.)
//
// What bounds it.  1024 frames x 32768 of 64 streams, 30 % of them skipped, 64
// taps, 7 powers: 320 us, from 745 us for v_mfma_f32_16x16x4_f32 over 16 x 16
// blocks of (phase, position) whose diagonals were added.  The samples alone
// take 80 us at the copy rate, the matrix core 160 us, the vector unit about
// as much (powers and their splits 40, rotations 30); two waves a SIMD overlap
// them in part.  301 frames of 255 to 20011 samples, banks of 8, 16 and 32
// taps, 10 powers: 34 us, from 98 us (each bank was summed by itself); the check
// of the sums takes 3 of them, 10 of the 320.  A run that is summed again takes
// 20 us and more, in which its workgroup does nothing else.
#include "bwd_common.h"
#include "runtime_kernels.h"
#include "split_common.h"

namespace prune {

namespace {
constexpr int kGhWaves = 4;
constexpr int kGhCh = 256;                  // input positions per chunk
constexpr int kGhBits = 15;                 // components are scaled below 2^15
constexpr float kGhMargin = 0x1p-8f;        // 2^17 times an operand's 2^-25
constexpr int kGhPow = 8;                   // powers per column group
constexpr int kGhUP = kGhCh + 4;            // words of a basis plane: rows of eight powers hit distinct banks
constexpr int kGhGP = kGhCh + PRUNE_MAX_L + 4;

struct GhWave {
  uint32_t u[2][kGhPow][kGhUP];             // [high, low][power][position]
  uint32_t g[2][kGhGP];
};
constexpr int kGhTot = 2 * PRUNE_MAX_L * 16;   // sums of a wave: [column group][tap][column]
constexpr int kGhErr = kGhTot;                 // and 2^17 T: [column group][column]
static_assert(sizeof(GhWave::u) >= (kGhTot + 32) * sizeof(float), "the sums fit in the basis planes");

// r^e for 0 <= e < 16 by binary powering, without branches.
__device__ __forceinline__ float ipow(float r, int e) {
  float p = 1.f, q = r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    p *= ((e >> k) & 1) ? q : 1.f;
    q *= q;
  }
  return p;
}

// Sums of a chunk by the fp32 definition, in the matrix-core layout:
// out[((group * 4 + row tile) * 64 + lane) * 4 + e].  in: re, im and magnitude
// of the chunk's samples, re and im of the cotangents (kGhCh and PRUNE_MAX_L
// more), zeros outside the frame.
constexpr int kGhIn = 3 * kGhCh + 2 * (kGhCh + PRUNE_MAX_L);
static_assert(sizeof(GhWave::u) >= (kGhIn + kGhTot) * sizeof(float), "a chunk and its sums fit in the basis planes");
template <int RT>
__device__ __noinline__ void gh_chunk_fp32(const float *in, float *out, int KH, int lane) {
  const int li = lane & 15, dp = lane >> 5, comp = (lane >> 4) & 1;
  const float *g = in + 3 * kGhCh + comp * (kGhCh + PRUNE_MAX_L);
  for (int grp = 0; 8 * grp < KH; ++grp) {
    const int power = 8 * grp + (li >> 1);
    floatx4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < kGhCh / 2; ++s) {
      const int p = 2 * s + dp;
      const float w = ipow(in[2 * kGhCh + p], power);
      const float ur = in[p] * w, ui = in[kGhCh + p] * w;
      const float b = power >= KH ? 0.f : (li & 1) ? (comp ? ur : -ui) : (comp ? ui : ur);
#pragma unroll
      for (int t = 0; t < RT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(g[p + 16 * t + li], b, acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) *(floatx4 *)(out + ((grp * 4 + t) * 64 + lane) * 4) = acc[t];
  }
}

// One column group of a chunk: nq times four steps.  gp: g's high plane at
// this lane's row and position group, up: the lane's power's high plane at
// the position group; rot, sgn turn (ur, ui) into (-ui, ur) for odd columns.
template <int RT>
__device__ __forceinline__ void gh_products(const uint32_t *gp, const uint32_t *up, int nq, uint32_t rot, uint32_t sgn,
                                            floatx4 (&acc)[RT]) {
  floatx4 low[RT], high[2][RT];   // two sums: half the roundings in each
#pragma unroll
  for (int t = 0; t < RT; ++t) high[0][t] = high[1][t] = low[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  half8 ah[RT + 3], al[RT + 3];
  auto row = [&](int i, int s) {
    ah[i] = __builtin_bit_cast(half8, *(const uintx4_u *)(gp + 16 * s));
    al[i] = __builtin_bit_cast(half8, *(const uintx4_u *)(gp + kGhGP + 16 * s));
  };
#pragma unroll
  for (int i = 0; i < RT - 1; ++i) row(i, i);
  for (int q = 0; q < nq; ++q) {
#pragma unroll
    for (int i = 0; i < 4; ++i) row(RT - 1 + i, 4 * q + RT - 1 + i);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uintx4 wh = *(const uintx4 *)(up + 64 * q + 16 * i), wl = *(const uintx4 *)(up + kGhPow * kGhUP + 64 * q + 16 * i);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        wh[k] = __builtin_amdgcn_alignbit(wh[k], wh[k], rot) ^ sgn;
        wl[k] = __builtin_amdgcn_alignbit(wl[k], wl[k], rot) ^ sgn;
      }
      const half8 bh = __builtin_bit_cast(half8, wh), bl = __builtin_bit_cast(half8, wl);
#pragma unroll
      for (int t = 0; t < RT; ++t) low[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[i + t], bh, low[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < RT; ++t)
        high[i & 1][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[i + t], bh, high[i & 1][t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < RT; ++t) low[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[i + t], bl, low[t], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < RT - 1; ++i) {
      ah[i] = ah[i + 4];
      al[i] = al[i + 4];
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = high[0][t] + (high[1][t] + low[t]);
}

// A wave's chunks w, w + 4, ... of a run: input positions [a0, pend) of frame
// F, RT row tiles of taps, KH powers, by the fp32 definition if `whole`.  The
// sums go to the wave's T, and after them 2^17 times what they may miss.
template <int RT>
__device__ __forceinline__ void gh_run(const BwdFrame &F, int a0, int pend, int KH, bool whole, GhWave &sh, int lane,
                                       int w) {
  asm volatile("" : "+v"(lane));
  const int n = (int)F.n, t0 = (int)F.t0;
  const int li = lane & 15, kg = lane >> 4;
  const uint32_t rot = (li & 1) ? 16u : 0u, sgn = (li & 1) ? 0x8000u : 0u;
  float neg1 = -1.f;
  asm volatile("" : "+v"(neg1));
  floatx4 tot[2][RT];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int t = 0; t < RT; ++t) tot[k][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  float err[2] = {0.f, 0.f};
  // lane l: positions 4 l .. 4 l + 3 of x and g, and position 256 + l of g
  pair_u xv[2], gv[2];
  float2 ge = make_float2(0.f, 0.f);
  auto load = [&](int a) {
    if (a >= 0 && a + kGhCh <= pend && a + kGhCh + PRUNE_MAX_L <= n) {   // uniform
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        xv[q] = ld_pair(F.x + a + 4 * lane + 2 * q);
        gv[q] = ld_pair(F.g + a + 4 * lane + 2 * q);
      }
      ge = ld_global(F.g + a + kGhCh + lane);
    } else {
      float2 xs[4], gs[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p = a + 4 * lane + q;
        xs[q] = p >= -t0 && p < pend ? ld_global(F.x + p) : make_float2(0.f, 0.f);
        gs[q] = p >= 0 && p < n ? ld_global(F.g + p) : make_float2(0.f, 0.f);
      }
      const int p = a + kGhCh + lane;
      ge = p < n && p >= 0 ? ld_global(F.g + p) : make_float2(0.f, 0.f);
      xv[0] = pair_u{xs[0].x, xs[0].y, xs[1].x, xs[1].y}; xv[1] = pair_u{xs[2].x, xs[2].y, xs[3].x, xs[3].y};
      gv[0] = pair_u{gs[0].x, gs[0].y, gs[1].x, gs[1].y}; gv[1] = pair_u{gs[2].x, gs[2].y, gs[3].x, gs[3].y};
    }
  };
  int a = a0 + kGhCh * w;
  if (a < pend) load(a);
  for (; a < pend; a += kGhCh * kGhWaves) {
    // scales and guards
    uint32_t xm = 0, gm = 0, gmin = ~0u;   // gmin: the least component of g that is not zero, less one
    float gsum = 0.f;
    auto take = [&](float v) {
      gm = max(gm, abs_bits(v));
      gmin = min(gmin, abs_bits(v) - 1u);
      gsum += fabsf(v);
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      xm = max(xm, max(max(abs_bits(xv[q].x), abs_bits(xv[q].y)), max(abs_bits(xv[q].z), abs_bits(xv[q].w))));
      take(gv[q].x); take(gv[q].y); take(gv[q].z); take(gv[q].w);
    }
    take(ge.x);
    take(ge.y);
    const uint32_t X = (uint32_t)wave_max((int)xm), G = (uint32_t)wave_max((int)gm);
    const bool bad = whole || (X != 0 && (X < kLow || X >= kHigh)) || (G != 0 && (G < kLow || G >= kHigh));
    if (!bad && (X == 0 || G == 0)) {
      if (a + kGhCh * kGhWaves < pend) load(a + kGhCh * kGhWaves);
      continue;
    }
    if (bad) {
      float *in = (float *)&sh.u[0][0][0], *out = in + kGhIn, *gp = in + 3 * kGhCh;
      wave_lds_fence();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const pair_u xq = xv[q >> 1], gq = gv[q >> 1];
        const float re = q & 1 ? xq.z : xq.x, im = q & 1 ? xq.w : xq.y;
        in[4 * lane + q] = re;
        in[kGhCh + 4 * lane + q] = im;
        in[2 * kGhCh + 4 * lane + q] = sqrtf(re * re + im * im);
        gp[4 * lane + q] = q & 1 ? gq.z : gq.x;
        gp[kGhCh + PRUNE_MAX_L + 4 * lane + q] = q & 1 ? gq.w : gq.y;
      }
      gp[kGhCh + lane] = ge.x;
      gp[kGhCh + PRUNE_MAX_L + kGhCh + lane] = ge.y;
      wave_lds_fence();
      gh_chunk_fp32<RT>(in, out, KH, lane);
      wave_lds_fence();
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (8 * k < KH) {
#pragma unroll
          for (int t = 0; t < RT; ++t) tot[k][t] += *(const floatx4 *)(out + ((k * 4 + t) * 64 + lane) * 4);
        }
      wave_lds_fence();
      if (a + kGhCh * kGhWaves < pend) load(a + kGhCh * kGhWaves);
      continue;
    }
    const int ex = (int)(X >> 23) - 126, eg = (int)(G >> 23) - 126;   // components < 2^ex, 2^eg
    // The matrix core drops the bits below its alignment towards minus
    // infinity, a small bias (0.06 of a step's rms error) that long sums would
    // collect: every other chunk is summed with the opposite sign.  Eight
    // powers, 16 taps, 524288 samples: 3.6e-7 without, 2.1e-7 with.
    const float flip = (a / (kGhCh * kGhWaves)) & 1 ? -1.f : 1.f;
    const float xs = __builtin_bit_cast(float, (uint32_t)(127 + kGhBits - ex) << 23) * flip;
    const float gs = __builtin_bit_cast(float, (uint32_t)(127 + kGhBits - eg) << 23);
    // components below one half (scaled; ten to a lane), and 2^17 T
    const uint32_t half = (uint32_t)max(126 + eg - kGhBits, 0) << 23;
    const float miss = kGhMargin * fmaf(wave_sum(gsum), gs, 0xap16f * (float)__popcll(__ballot(gmin < half)));
    // |x| as rho + rlo: a power's error would otherwise be |x|'s rounding, p
    // times, in the few largest samples that make up the sums of high powers
    pair_u v[2];
    float rho[4], rlo[4];
    uint32_t top = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      v[q] = xv[q] * xs;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float re = k ? v[q].z : v[q].x, im = k ? v[q].w : v[q].y;
        const float h2 = re * re, s2 = fmaf(im, im, h2), es = fmaf(im, im, h2 - s2) + fmaf(re, re, -h2);
        top = max(top, __builtin_bit_cast(uint32_t, s2));
        const float y = __builtin_amdgcn_rsqf(fmaxf(s2, 1e-30f)), r0 = s2 * y;
        const float c = (fmaf(-r0, r0, s2) + es) * (0.5f * y), r = r0 + c;
        rho[2 * q + k] = r * (1.f / (1 << kGhBits));
        rlo[2 * q + k] = (c - (r - r0)) * (1.f / (1 << kGhBits));
      }
    }
    // Power p is scaled up by 2^kp, so that its largest sample, |v| rho^p, lies
    // near 2^15 too (no component reaches half precision's 65504).
    const float lv =
        0.5f * __builtin_amdgcn_logf(fmaxf(__builtin_bit_cast(float, (uint32_t)wave_max((int)top)), 0x1p28f));
    auto lift = [&](int p) { return p ? (int)floorf(15.9f - lv - (float)p * (lv - kGhBits)) : 0; };
    const int kp = lift(lane & 15);
    wave_lds_fence();   // the last chunk's reads end here
    {
      uint32_t hi[4], lo[4];
      split_pair(gv[0] * gs, neg1, hi, lo);
      split_pair(gv[1] * gs, neg1, hi + 2, lo + 2);
      *(uintx4 *)&sh.g[0][4 * lane] = uintx4{hi[0], hi[1], hi[2], hi[3]};
      *(uintx4 *)&sh.g[1][4 * lane] = uintx4{lo[0], lo[1], lo[2], lo[3]};
      split_pair(pair_u{ge.x * gs, ge.y * gs, 0.f, 0.f}, neg1, hi, lo);
      sh.g[0][kGhCh + lane] = hi[0];
      sh.g[1][kGhCh + lane] = lo[0];
    }
    if (a + kGhCh * kGhWaves < pend) load(a + kGhCh * kGhWaves);   // in flight during the products
    const int nq = (min(kGhCh, pend - a) + 63) / 64;
    const uint32_t *gp = &sh.g[0][4 * kg + li], *up = &sh.u[0][li >> 1][4 * kg];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (8 * k >= KH) continue;
      if (k) wave_lds_fence();
      const int np = min(kGhPow, KH - 8 * k);
      for (int j = 0; j < np; ++j) {
        uint32_t hi[4], lo[4];
        split_pair(v[0], neg1, hi, lo);
        split_pair(v[1], neg1, hi + 2, lo + 2);
        *(uintx4 *)&sh.u[0][j][4 * lane] = uintx4{hi[0], hi[1], hi[2], hi[3]};
        *(uintx4 *)&sh.u[1][j][4 * lane] = uintx4{lo[0], lo[1], lo[2], lo[3]};
        const int p = 8 * k + j;
        const float sc = __builtin_bit_cast(
            float, (uint32_t)(127 + __builtin_amdgcn_readlane(kp, p + 1) - __builtin_amdgcn_readlane(kp, p)) << 23);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float h0 = rho[2 * q] * sc, l0 = rlo[2 * q] * sc, h1 = rho[2 * q + 1] * sc, l1 = rlo[2 * q + 1] * sc;
          v[q].x = fmaf(v[q].x, h0, v[q].x * l0);
          v[q].y = fmaf(v[q].y, h0, v[q].y * l0);
          v[q].z = fmaf(v[q].z, h1, v[q].z * l1);
          v[q].w = fmaf(v[q].w, h1, v[q].w * l1);
        }
      }
      wave_lds_fence();
      floatx4 acc[RT];
      gh_products<RT>(gp, up, nq, rot, sgn, acc);
      const int p = 8 * k + (li >> 1), sc = eg + ex - 2 * kGhBits + p * ex - lift(p);
      err[k] += ldexpf(miss, sc);
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tot[k][t][e] = fmaf(ldexpf(acc[t][e], sc), flip, tot[k][t][e]);
    }
  }
  wave_lds_fence();
  float *T = (float *)&sh.u[0][0][0];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) T[(k * PRUNE_MAX_L + 16 * t + 4 * kg + e) * 16 + li] = tot[k][t][e];
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (lane < 16) T[kGhErr + 16 * k + li] = err[k];
}
}  // namespace

// grad_h partials.  Work: runs of up to bwd_run_len consecutive tiles of one
// frame (item groups [g*run, g*run+run) split where the frame changes), four waves
// a run.  A run's sum is the partial row of its first item; the other items'
// rows are not written (bwd_run_row).
__global__ __launch_bounds__(64 * kGhWaves, 2) void k_bwd_gh_split(prune_fb_desc d, const BwdFrame *__restrict__ bf,
                                                                   const WorkItem *__restrict__ items,
                                                                   const uint32_t *__restrict__ n_items,
                                                                   unsigned int *__restrict__ ticket,
                                                                   float2 *__restrict__ partial) {
  __shared__ GhWave s_w[kGhWaves];
  __shared__ uint32_t s_grp, s_low[2];   // s_low: a sum of this attempt, of the next, is too small
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t Lmax = 1;
  for (uint32_t b = 0; b < d.n_banks; ++b) Lmax = max(Lmax, d.L[b]);
  const uint32_t E = d.n_banks * d.Kmax * Lmax;
  const uint32_t ni = *n_items;
  const uint32_t run = bwd_run_len(ni, gridDim.x), ng = (ni + run - 1) / run;
  const uint32_t kfull = (1u << d.Kmax) - 1u;
  uint32_t par = 0;
  if (t < 2) s_low[t] = 0;
  bool first = true;   // first run group by workgroup index, later ones by ticket
  for (;;) {
    if (t == 0) s_grp = first ? blockIdx.x : gridDim.x >= ng ? ng : gridDim.x + atomicAdd(ticket, 1u);
    first = false;
    __syncthreads();
    const uint32_t grp = s_grp;
    __syncthreads();   // s_grp is rewritten by the next ticket
    if (grp >= ng) break;
    const uint32_t i1 = min(ni, (grp + 1) * run);
    for (uint32_t r0 = grp * run; r0 < i1;) {
      // the run's items at once, a lane each (run <= 8)
      const WorkItem wi = items[min(r0 + (lane & 7), i1 - 1)];
      WorkItem w0;
      w0.frame = (uint32_t)__builtin_amdgcn_readfirstlane((int)wi.frame);
      w0.tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)wi.tile);
      const uint32_t other = ((uint32_t)__ballot(wi.frame != w0.frame) & 0xffu) | 1u << (i1 - r0);
      const uint32_t r1 = r0 + __ffs(other) - 1;
      const BwdFrame F = bf[w0.frame];
      float2 *row = partial + (size_t)r0 * E;
      uint32_t pm = 0, L = 0;
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        const uint32_t bm = F.route ? 0u : (F.mask >> (bank * d.Kmax)) & kfull;
        pm |= bm;
        if (bm) L = max(L, d.L[bank]);
      }
      // input positions: this run's samples, and the history of the frame's first tile
      const int n = (int)F.n, a0 = w0.tile ? (int)w0.tile * kBT : (L > 1 ? -PRUNE_MAX_L : 0);
      // taps that reach beyond the frame from all of them have no term
      const int reach = n - max(a0, -(int)F.t0);
      for (bool whole = false;;) {
        if (pm) {
          const int KH = 32 - __clz(pm);
          const int pend = min(n, ((int)w0.tile + (int)(r1 - r0)) * kBT);
          if (L <= 16) gh_run<1>(F, a0, pend, KH, whole, s_w[w], lane, w);
          else if (L <= 32) gh_run<2>(F, a0, pend, KH, whole, s_w[w], lane, w);
          else if (L <= 48) gh_run<3>(F, a0, pend, KH, whole, s_w[w], lane, w);
          else gh_run<4>(F, a0, pend, KH, whole, s_w[w], lane, w);
        }
        __syncthreads();
        bool low = false;
        for (uint32_t k = t; k < E; k += 64 * kGhWaves) {
          const uint32_t br = k / Lmax, l = k - br * Lmax, bank = br / d.Kmax, p = br - bank * d.Kmax;
          float2 v = make_float2(0.f, 0.f);
          if (pm && ((F.mask >> br) & 1u) && l < d.L[bank]) {
            float miss = 0.f;
#pragma unroll
            for (int q = 0; q < kGhWaves; ++q) {
              const float *T = (const float *)&s_w[q].u[0][0][0], *c = T + ((p >> 3) * PRUNE_MAX_L + l) * 16 + 2 * (p & 7);
              v.x += c[0];
              v.y += c[1];
              miss += T[kGhErr + 16 * (p >> 3) + 2 * (p & 7)];
            }
            low |= (int)l < reach && fmaxf(fabsf(v.x), fabsf(v.y)) < miss;
          }
          row[k] = v;
        }
        if (low) s_low[par] = 1u;
        if (t == 0) s_low[par ^ 1u] = 0u;
        __syncthreads();   // the LDS is rewritten, by the run again or the next one
        whole = !whole && __builtin_amdgcn_readfirstlane((int)s_low[par]);
        par ^= 1u;
        if (!whole) break;
      }
      r0 = r1;
    }
  }
}

void launch_bwd_gh_split(const prune_fb_desc &d, const BwdFrame *bf, const WorkItem *items,
                         const uint32_t *n_items, unsigned int *ticket, float2 *partial, uint32_t grid,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_bwd_gh_split, dim3(grid), dim3(64 * kGhWaves), 0, s, d, bf, items, n_items, ticket, partial);
}

}  // namespace prune
