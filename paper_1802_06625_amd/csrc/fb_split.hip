// Filter-bank forward on the half-precision matrix cores with split operands:
// the block-Toeplitz form of the fused basis + FIR + branch-sum firing
// (Sec. VII-A), for filters of 25 to 64 taps.
//
// An output block of 16 samples from q on is, per power p of its basis
// u_p = |x|^p x,
//   y[q + i] += sum_m h_p[i + HOFF - m] u_p[q - HOFF + m],   m < 8 S, HOFF = 8 S - 16,
// a product of the Toeplitz matrix of the taps (32 rows: 16 phases x re, im;
// contraction: 8 S positions x re, im) with the Hankel matrix of the samples
// (columns: blocks), on v_mfma_f32_32x32x16_f16 in S steps of 8 positions.
//
// Precision.  Every fp32 operand is the sum of two half-precision parts,
// v = high + low, after a scaling by powers of two: each power of the samples
// of a wave's window so that the largest lies near 2^15, the taps of each
// power so that the largest lies in [2^14, 2^15).  The products high x high,
// low x high and high x low are exact in the fp32 accumulators; low x low
// (2^-24 of the product) is left out.  The matrix core rounds its sum once
// per eight terms, so each power is summed in accumulators of its own, low
// products first, and added to the running sum in fp32.  Relative error
// against fp64 for 25 to 64 taps, 1 to 10 branches, Gaussian and
// constant-envelope samples: 1.0e-7 to 1.6e-7 (up to 3.5e-7 where |x|^9
// dominates), at or below the vector kernels' 1.3e-7 to 2.1e-7 (3.5e-7);
// below 25 taps the vector kernels are the more exact, so the autotuner
// offers these only where every bank has kSplitMinTaps.
//
// The two parts keep an operand to 2^-23 of itself down to 2^-2, and to 2^-25
// at any size below, which is 2^-40 of its power's largest in the window.  An
// output may depend on such operands alone (a quiet stretch beside a loud one,
// where a high power of the quiet samples is far below the window's, or taps
// that leave out the loud samples), so the parts that can be missing are
// bounded and compared with the outputs themselves: with HS_p the sum of the
// magnitudes of power p's scaled taps (and 2^16 for each tap component below
// one half), no component of an output misses more than T = 2^-25 sum_p HS_p
// of the powers' sums (its rms is a tenth of that or less).  Outputs below
// 2^17 T are evaluated one by one in fp32 instead; a wave that has more than
// kFew of them, or a lane with all of its outputs (sixteen of 32 in a row)
// below 2^20 T, evaluates all of its outputs so, and a wave whose samples or
// taps are not finite or beyond 2^93.  Outputs of windows of zeros are exact
// zeros and stay.  Gaussian samples and taps have their outputs' median at
// 2^30 T (ten powers, |x|^9 in front: one wave in 300 has an output below
// 2^17 T) to 2^33 T.
//
// Work.  A work item is TILE outputs of one frame, done in passes of 4 waves
// x 512 NT outputs (NT = 2, 1 for a frame's last 2048).  A wave keeps its
// window in registers (two samples a lane and run of 128), multiplies it by
// |x| from power to power, and writes the two parts of each power to its own
// LDS planes, from which the column operands are read: 16-byte chunks of four
// (re, im) pairs, one pad chunk per column so that sixteen lanes' reads hit
// distinct banks.  The tap table of a bank (all powers, both parts, reversed
// so that a Toeplitz row is a run of words) is kept in LDS while frames share
// it.  No barrier inside a pass; the next pass's window is loaded during the
// last power's products.
//
// What bounds it.  4096 frames x 16384, 1..10 branches, 32 taps: 540-560 us
// against 740-765 us for the vector kernel at 64 % of its FMA ceiling.  Of
// that, the 1.07 GB of samples take 230 us at the copy rate, the matrix core
// 215 us (39 %), the vector unit about 210 us (basis, split, sums) and the
// LDS about 250 us; two waves a SIMD overlap them only in part.  33.5M samples
// with 64 taps and 7 branches: 420 us against 740 us.
// Measured without gain: four result tiles a wave at one wave a SIMD (689
// us), three waves a SIMD (spills, 1070 us), the window loaded a whole pass
// ahead (557 us), vector work placed between the products by hand (640 us).
#include <hip/hip_ext.h>

#include <type_traits>

#include "prune_internal.h"
#include "runtime_kernels.h"
#include "split_common.h"

namespace prune {

namespace {
constexpr int kSplitWaves = 4;                   // waves of a workgroup
constexpr int kSplitPow = 10;                    // powers of a bank
constexpr int kSplitTab = PRUNE_MAX_L + 32;      // table entries per power: 8 S + 16 at most
constexpr int kTapBits = 15, kSampleBits = 15;   // the largest tap and the largest component are scaled below 2^15
constexpr float kSplitMargin = 0x1p-8f;          // 2^17 times an operand's 2^-25

// Frame descriptors and work items are constant while the kernel runs and
// the same for a whole workgroup: read through the scalar cache.
typedef const __attribute__((address_space(4))) FbFrameDesc CDesc;
typedef const __attribute__((address_space(4))) WorkItem CItem;

struct SplitShared {
  uint32_t tab[kSplitPow][2][2][kSplitTab];   // [power][high, low part][re, im row][reversed tap]
  int cexp[16];                               // per power: its largest tap is below 2^cexp
  int hsum[16];                               // per power: HS_p
  uint32_t next[2];
};
constexpr int kNoTap = -100000, kBadTap = 100000;
constexpr float kHuge = 3e38f;
// LDS word of window sample 2 lane + 128 i: one pad chunk of four samples per
// column of 16 NT samples (a power of two up to 64).
template <int NT>
__device__ __forceinline__ int plane_idx(int lane, int i) {
  return 2 * lane + 4 * (2 * lane / (16 * NT)) + (128 + 4 * (8 / NT)) * i;
}

// Words of one operand plane of a wave: window samples in whole runs of 128,
// and the pads.
constexpr int split_plane(int nt) { return (4 * nt + 1) * (128 + 4 * (8 / nt)); }

// The wave's window of a pass of 4 x 512 nt outputs from frame position n0
// on: kHist samples before its first output, then its outputs' samples; lane
// l holds samples 2 l + 128 i and the next one.
constexpr int kHist = 64;
__device__ __forceinline__ bool window_inside(CDesc &d, int wb, int nt) {
  return wb >= kHist && wb + 512 * nt + 64 <= (int)d.n;
}

// A pass's window as the loads need it: null unless the pass is of the largest
// size and the window lies inside the frame.
template <int NTMAX>
__device__ __forceinline__ const float2 *window_ptr(CDesc &d, int n0, int nt, int w) {
  const int wb = n0 + w * 512 * nt;
  return nt == NTMAX && window_inside(d, wb, nt) ? d.x + (wb - kHist) : nullptr;
}

// Loads only, in flight until v is used.
template <int NTMAX>
__device__ __forceinline__ void prefetch_window(const float2 *x, int lane, pair_u *v) {
  constexpr int NP = 4 * NTMAX + 1;
  // v's old values end here: the loads take their registers
#pragma unroll
  for (int i = 0; i < NP; ++i) asm volatile("" : "=v"(v[i]));
  if (x) {
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = ld_pair(x + 2 * lane + 128 * i);
  }
}

// Windows that reach past the frame: its halo before it, zeros after it.
template <int NP>
__device__ __forceinline__ void load_edge(CDesc &d, int wb, int lane, pair_u *v) {
  const float2 *halo = d.halo + ((int)d.Lmax - 1);
  const int n = (int)d.n, hv = (int)d.halo_valid, p0 = wb - kHist + 2 * lane;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    float2 z[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int p = p0 + 128 * i + q;
      z[q] = make_float2(0.f, 0.f);
      if (p >= 0 ? p < n : -p <= hv) z[q] = ld_global((p >= 0 ? d.x : halo) + p);
    }
    v[i] = pair_u{z[0].x, z[0].y, z[1].x, z[1].y};
  }
}

// The tap table of one frame: every power of its bank when a single bank is
// active, the sums over the banks of its mask's branches otherwise.
template <int S>
__device__ __forceinline__ void build_table(CDesc &d, int bank1, SplitShared &sh) {
  constexpr int TS = 8 * S + 16, NE = (kSplitPow * TS + 255) / 256;
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  float2 h[NE];
  if (t < 16) {
    sh.cexp[t] = kNoTap;
    sh.hsum[t] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int k = t + 256 * i, p = k / TS, l = 8 * S - 1 - (k - p * TS);
    h[i] = make_float2(0.f, 0.f);
    if (p < (int)d.Kmax && l >= 0) {
      for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
        const bool on = bank1 >= 0 ? (int)bank == bank1 : ((d.mask >> (bank * d.Kmax + p)) & 1u) != 0;
        if (on && l < (int)d.L[bank]) {
          const float2 z = ld_global(d.taps + (size_t)(bank * d.Kmax + p) * d.Lmax + l);
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
  for (int i = 0; i < NE; ++i) {
    const int k = t + 256 * i, p = k / TS, q = k - p * TS;
    if (p < kSplitPow) {
      const int sc = kTapBits - sh.cexp[p];
      const float hr = ldexpf(h[i].x, sc), hi = ldexpf(h[i].y, sc), ar = fabsf(hr), ai = fabsf(hi);
      if (ar + ai > 0.f && sh.cexp[p] != kBadTap)
        atomicAdd(&sh.hsum[p], (int)ceilf(ar + ai) + (ar > 0.f && ar < 0.5f ? 1 << 16 : 0) +
                                   (ai > 0.f && ai < 0.5f ? 1 << 16 : 0));
      const _Float16 r1 = (_Float16)hr, i1 = (_Float16)hi;
      const _Float16 r2 = (_Float16)(hr - (float)r1), i2 = (_Float16)(hi - (float)i1);
      sh.tab[p][0][0][q] = __builtin_bit_cast(uint32_t, half2v{r1, (_Float16)-i1});
      sh.tab[p][0][1][q] = __builtin_bit_cast(uint32_t, half2v{i1, r1});
      sh.tab[p][1][0][q] = __builtin_bit_cast(uint32_t, half2v{r2, (_Float16)-i2});
      sh.tab[p][1][1][q] = __builtin_bit_cast(uint32_t, half2v{i2, r2});
    }
  }
  __syncthreads();
}

// Taps 0 .. L - 1 of KH powers (lane l holds taps l, so that a tap is a scalar
// when its turn comes) against a window in the planes: eight outputs a lane.
constexpr int kF32J = 8, kF32Win = kHist + 64 * kF32J, kF32Plane = kF32Win + kF32Win / kF32J;
template <int KH>
__device__ __forceinline__ void fp32_taps(const float *plane, int lane, int L, const float2 *tap, float *yr, float *yi) {
  constexpr int J = kF32J, CH = 8;             // taps per register window
  auto scalar = [](float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  };
  for (int l0 = 0; l0 < L; l0 += CH) {
    // window sample w is stream position (first output) - l0 - (CH - 1) + w
    float xr[J + CH - 1], xi[J + CH - 1], r[J + CH - 1];
#pragma unroll
    for (int w = 0; w < J + CH - 1; ++w) {
      const int k = kHist + J * lane - l0 - (CH - 1) + w, a = k + k / J;
      xr[w] = plane[a];
      xi[w] = plane[kF32Plane + a];
      r[w] = plane[2 * kF32Plane + a];
    }
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      if (l0 + i >= L) break;
      float ar[J], ai[J];
#pragma unroll
      for (int b = KH - 1; b >= 0; --b) {
        const float cx = scalar(tap[b].x, l0 + i), cy = scalar(tap[b].y, l0 + i);
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int w = j - i + CH - 1;
          ar[j] = b == KH - 1 ? cx : fmaf(ar[j], r[w], cx);
          ai[j] = b == KH - 1 ? cy : fmaf(ai[j], r[w], cy);
        }
      }
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int w = j - i + CH - 1;
        yr[j] = fmaf(xr[w], ar[j], yr[j]);
        yr[j] = fmaf(-xi[w], ai[j], yr[j]);
        yi[j] = fmaf(xr[w], ai[j], yi[j]);
        yi[j] = fmaf(xi[w], ar[j], yi[j]);
      }
    }
  }
}

// 512 of a wave's outputs by the fp32 definition (the vector kernels' Horner
// form, eight outputs a lane), for waves that the scaled split cannot take.
// 1024 x 16384, ten branches, 32 taps, every wave here after its passes: 677 us
// (221 without; the vector kernel 292).  Not inlined: its registers would cost
// the passes theirs (spills, 517 -> 600 us on the 4096 x 16384 batch).
__device__ __noinline__ void fp32_outputs(CDesc &d, int wb, float *plane, int lane) {
  constexpr int J = kF32J;
  const float2 *halo = d.halo + ((int)d.Lmax - 1);
  const int n = (int)d.n, hv = (int)d.halo_valid;
  const uint32_t kfull = (1u << d.Kmax) - 1u;
  float2 z[kF32Win / 64];
#pragma unroll
  for (int i = 0; i < kF32Win / 64; ++i) {
    const int p = wb - kHist + lane + 64 * i;
    z[i] = make_float2(0.f, 0.f);
    if (p >= 0 ? p < n : -p <= hv) z[i] = ld_global((p >= 0 ? d.x : halo) + p);
  }
  wave_lds_fence();
#pragma unroll
  for (int i = 0; i < kF32Win / 64; ++i) {
    const int k = lane + 64 * i, a = k + k / J;
    plane[a] = z[i].x;
    plane[kF32Plane + a] = z[i].y;
    plane[2 * kF32Plane + a] = magnitude(z[i].x, z[i].y);
  }
  wave_lds_fence();
  float yr[J], yi[J];
#pragma unroll
  for (int j = 0; j < J; ++j) yr[j] = yi[j] = 0.f;
  for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
    const uint32_t bmask = (d.mask >> (bank * d.Kmax)) & kfull;
    if (!bmask) continue;
    const int KH = 32 - __clz(bmask), L = (int)d.L[bank];
    const float2 *tb = d.taps + (size_t)bank * d.Kmax * d.Lmax;
    float2 tap[kSplitPow];
#pragma unroll
    for (int b = 0; b < kSplitPow; ++b) {
      tap[b] = make_float2(0.f, 0.f);
      if (((bmask >> b) & 1u) && lane < L) tap[b] = ld_global(tb + (size_t)b * d.Lmax + lane);
    }
    switch (KH) {
#define PRUNE_FP(k) case k: fp32_taps<k>(plane, lane, L, tap, yr, yi); break
      PRUNE_FP(1); PRUNE_FP(2); PRUNE_FP(3); PRUNE_FP(4); PRUNE_FP(5);
      PRUNE_FP(6); PRUNE_FP(7); PRUNE_FP(8); PRUNE_FP(9);
      default: fp32_taps<10>(plane, lane, L, tap, yr, yi);
#undef PRUNE_FP
    }
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int p = wb + J * lane + j;
    if (p < n)
      for (uint32_t o = 0; o < d.n_y; ++o) st_global(d.y[o] + p, make_float2(yr[j], yi[j]));
  }
  wave_lds_fence();
}

// A lane's output b of a wave (in the order of split_pass): its place from wb.
template <int NT>
__device__ __forceinline__ int output_at(int lane, int b) {
  return 16 * NT * (lane & 31) + 2 * (lane >> 5) + 16 * (b >> 3) + 4 * ((b >> 1) & 3) + (b & 1);
}

// The outputs in `few` (a bit for each of the lane's) by the fp32 definition,
// one after another, a lane for each tap.
template <int NT>
__device__ __noinline__ void fix_outputs(CDesc &d, int wb, uint32_t few, int lane) {
  const float2 *halo = d.halo + ((int)d.Lmax - 1);
  const int hv = (int)d.halo_valid;
  const uint32_t kfull = (1u << d.Kmax) - 1u;
  for (;;) {
    const unsigned long long who = __ballot(few != 0u);
    if (!who) break;
    const int src = __ffsll(who) - 1, b = __ffs(__builtin_amdgcn_readlane((int)few, src)) - 1;
    const int at = wb + output_at<NT>(src, b), p = at - lane;
    float2 z = make_float2(0.f, 0.f);
    if (p >= 0 || -p <= hv) z = ld_global((p >= 0 ? d.x : halo) + p);
    const float r = magnitude(z.x, z.y);
    float yr = 0.f, yi = 0.f;
    for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
      const uint32_t bmask = (d.mask >> (bank * d.Kmax)) & kfull;
      if (!bmask) continue;
      const float2 *tb = d.taps + (size_t)bank * d.Kmax * d.Lmax;
      const bool on = lane < (int)d.L[bank];
      float ar = 0.f, ai = 0.f;
      for (int k = 31 - __clz(bmask); k >= 0; --k) {
        const float2 c = on && ((bmask >> k) & 1u) ? ld_global(tb + (size_t)k * d.Lmax + lane) : make_float2(0.f, 0.f);
        ar = fmaf(ar, r, c.x);
        ai = fmaf(ai, r, c.y);
      }
      if (on) {
        yr += fmaf(z.x, ar, -z.y * ai);
        yi += fmaf(z.x, ai, z.y * ar);
      }
    }
    for (int o = 32; o; o >>= 1) {
      yr += __shfl_xor(yr, o, 64);
      yi += __shfl_xor(yi, o, 64);
    }
    if (lane < (int)d.n_y) st_global(d.y[lane] + at, make_float2(yr, yi));
    if (lane == src) few &= few - 1u;
  }
}

// Whether the windows of L samples of the outputs in `zeros` (a bit for each of
// the lane's) hold zeros only.
template <int NT>
__device__ __noinline__ bool silent_windows(CDesc &d, int wb, int L, uint32_t zeros, uint32_t *plane, int lane) {
  const float2 *halo = d.halo + ((int)d.Lmax - 1);
  const int n = (int)d.n, hv = (int)d.halo_valid;
  const unsigned long long lt = (1ull << lane) - 1ull, le = lt | 1ull << lane;
  auto top = [](unsigned long long m) { return m ? 63 - __clzll((long long)m) : -(1 << 20); };
  int last = -(1 << 20);                       // the last sample before this run that is not zero
  wave_lds_fence();
  for (int i = 0; i < 4 * NT + 1; ++i) {
    unsigned long long on[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int p = wb - kHist + 2 * lane + 128 * i + q;
      float2 z = make_float2(0.f, 0.f);
      if (p >= 0 ? p < n : -p <= hv) z = ld_global((p >= 0 ? d.x : halo) + p);
      on[q] = __ballot((abs_bits(z.x) | abs_bits(z.y)) != 0u);
    }
    const int k = 128 * i, even = 2 * top(on[0] & le);
    plane[k + 2 * lane] = (uint32_t)max(last, k + max(even, 2 * top(on[1] & lt) + 1));
    plane[k + 2 * lane + 1] = (uint32_t)max(last, k + max(even, 2 * top(on[1] & le) + 1));
    last = max(last, k + max(2 * top(on[0]), 2 * top(on[1]) + 1));
  }
  wave_lds_fence();
  bool ok = true;
  for (int b = 0; b < 8 * NT; ++b) {
    const int k = kHist + output_at<NT>(lane, b);
    if ((zeros >> b) & 1u) ok &= k - (int)plane[k] >= L;
  }
  wave_lds_fence();
  return !__any(!ok);
}

// One pass: 4 waves x 32 columns x 16 NT outputs from frame position n0 on.
// x holds the wave's window if the pass is of the largest size and the window
// lies inside the frame; prefetch() issues the loads of the next pass's.
// kPassLeft: nothing is written, the wave's outputs are left to the fp32
// definition.  kPassCheck: everything is written; the outputs in the upper half
// of `flags` (a bit for each of the lane's) are to be evaluated again, and where
// the window of one in the lower half does not hold zeros only
// (silent_windows), all of the wave's are.
enum { kPassDone, kPassLeft, kPassCheck };
constexpr int kFew = 12;
template <int NT, int S, int NTMAX, class Prefetch>
__device__ __forceinline__ int split_pass(CDesc &d, int n0, uint32_t pm, const SplitShared &sh,
                                          uint32_t *__restrict__ plane, pair_u *x, int lane, int w,
                                          uint32_t &flags, const Prefetch &prefetch) {
  constexpr int HOFF = 8 * S - 16;             // window samples that an output block reads before itself
  constexpr int C0 = (kHist - HOFF) / 4;       // window chunks (of 4 samples) before those
  constexpr int NP = 4 * NT + 1;               // sample pairs per lane
  constexpr int NC = 2 * NT + S - 2;           // chunks per lane
  constexpr int PLANE = split_plane(NTMAX);
  // opaque to the compiler, which would otherwise keep every lane-dependent
  // address of every instantiation across the persistent loop, in scratch
  asm volatile("" : "+v"(lane));
  const int n = (int)d.n, wb = n0 + w * 512 * NT;
  if (wb >= n) {
    prefetch();
    return kPassDone;
  }
  if (NT < NTMAX || !window_inside(d, wb, NT)) load_edge<NP>(d, wb, lane, x);
  float am = 0.f;                              // largest |re|, |im| (NaN left out)
#pragma unroll
  for (int i = 0; i < NP; ++i)
    am = fmaxf(fmaxf(am, fmaxf(fabsf(x[i].x), fabsf(x[i].y))), fmaxf(fabsf(x[i].z), fabsf(x[i].w)));
  const uint32_t A = (uint32_t)wave_max(__builtin_bit_cast(int, am));
  const int e = A >= kLow ? (int)(A >> 23) - 126 : 0;   // |re|, |im| < 2^e
  const int li = lane & 31, g = lane >> 5;
  pair_u v[NP];                                // the current power of the samples, scaled
  float rho[NP][2], neg1 = -1.f;               // |x| / 2^e
  asm volatile("" : "+v"(neg1));
  uint32_t top = 0;
  {
    const float xs = __builtin_bit_cast(float, (uint32_t)(127 + kSampleBits - e) << 23);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      v[i] = x[i] * xs;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float a = q ? v[i].z : v[i].x, b = q ? v[i].w : v[i].y;
        const float s2 = fmaf(a, a, b * b);
        top = max(top, __builtin_bit_cast(uint32_t, s2));
        const float y = __builtin_amdgcn_rsqf(fmaxf(s2, 1e-30f));
        const float r0 = s2 * y;
        rho[i][q] = fmaf(fmaf(-r0, r0, s2), 0.5f * y, r0) * (1.f / (1 << kSampleBits));
      }
    }
  }
  const uint32_t S2 = (uint32_t)wave_max((int)min(top, kInf));   // |v|^2 of the largest, or a NaN sample
  // Power p is scaled up by 2^kp, so that its largest sample, |v| rho^p, lies
  // near 2^15 too (no component reaches half precision's 65504).
  const float lv = 0.5f * __builtin_amdgcn_logf(fmaxf(__builtin_bit_cast(float, S2), 0x1p28f));
  const int kp = lane && lane < kSplitPow ? (int)floorf(15.9f - lv - (float)lane * (lv - kSampleBits)) : 0;
  // power p's products carry 2^-(ep - kTapBits - kSampleBits); they are added
  // up relative to the largest of the active powers
  int ep = kNoTap;
  if (lane < kSplitPow && ((pm >> lane) & 1u)) ep = sh.cexp[lane];
  if (__any(ep == kBadTap) || (A != 0 && (A < kLow || A >= kHigh)) || S2 >= kInf) return kPassLeft;
  ep += lane * e - kp;
  const int eb = wave_max(ep);
  const float ef = ldexpf(1.f, max(ep - eb, -200));
  const float hs = kSplitMargin * (float)sh.hsum[lane & 15];
  // what an output has to reach; at least 2^-80, so that no power that is
  // missing for its ef counts (silence and zero taps give exact zeros)
  float thr = A == 0 || eb < kNoTap / 2 ? 0.f : 0x1p-80f;
  auto uniform = [](float f, int p) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f), p));
  };
  auto scale_to = [&](int p) {                 // from power p - 1 to power p
    const int k = __builtin_amdgcn_readlane(kp, p) - __builtin_amdgcn_readlane(kp, p - 1);
    return __builtin_bit_cast(float, (uint32_t)(127 + k) << 23);
  };
  auto advance = [&](int i, float sc) {
    const float r0 = rho[i][0] * sc, r1 = rho[i][1] * sc;
    v[i].x *= r0; v[i].y *= r0;
    v[i].z *= r1; v[i].w *= r1;
  };
  auto put = [&](int i) {
    uint32_t hi[2], lo[2];
    split_pair(v[i], neg1, hi, lo);
    const int q = plane_idx<NT>(lane, i);
    *(uintx2 *)(plane + q) = uintx2{hi[0], hi[1]};
    *(uintx2 *)(plane + PLANE + q) = uintx2{lo[0], lo[1]};
  };
  floatx16 tot[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) tot[j][q] = 0.f;
  const uint32_t *trow = &sh.tab[0][0][li & 1][15 - (li >> 1) + 4 * g];
  constexpr int CW = 4 * NT;                   // chunks per column
  const uint32_t *brow = plane + (CW + 1) * 4 * li + 4 * g;
  // One power: its products, and the next power's operands
  auto power = [&](int p, int next, auto last) {
    const uint32_t *tp = trow + p * (4 * kSplitTab);
    floatx16 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
    // Even chunks meet the even steps of the taps and odd ones the odd steps:
    // half of the operands are in registers at a time.  Of each half the
    // products of the low parts come first, while the sum is small.
    half8 ah[S], al[S], bh[NC], bl[NC];
    auto fetch = [&](int odd) {
#pragma unroll
      for (int s = odd; s < S; s += 2) {
        ah[s] = __builtin_bit_cast(half8, *(const uintx4_u *)(tp + 8 * s));
        al[s] = __builtin_bit_cast(half8, *(const uintx4_u *)(tp + 2 * kSplitTab + 8 * s));
      }
#pragma unroll
      for (int i = odd; i < NC; i += 2) {
        const int o = 4 * (C0 + 2 * i + (C0 + 2 * i) / CW);
        bh[i] = __builtin_bit_cast(half8, *(const uintx4 *)(brow + o));
        bl[i] = __builtin_bit_cast(half8, *(const uintx4 *)(brow + PLANE + o));
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
    auto low = [&](int odd) {
      mma(odd, al, bh);
      mma(odd, ah, bl);
    };
    fetch(0);
    low(0);
    mma(0, ah, bh);
    fetch(1);
    wave_lds_fence();
    if (!decltype(last)::value) {
      const float sc = scale_to(next);
#pragma unroll
      for (int i = 0; i < NP; ++i) { advance(i, sc); put(i); }
    }
    low(1);
    mma(1, ah, bh);
    const float f = uniform(ef, p);
    if (thr > 0.f) thr = fmaf(f, uniform(hs, p), thr);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) tot[j][q] = fmaf(acc[j][q], f, tot[j][q]);
    wave_lds_fence();
  };
  int p = 0;
  for (; !((pm >> p) & 1u); ++p) {
    const float sc = scale_to(p + 1);
#pragma unroll
    for (int i = 0; i < NP; ++i) advance(i, sc);
  }
  wave_lds_fence();
#pragma unroll
  for (int i = 0; i < NP; ++i) put(i);
  wave_lds_fence();
  for (uint32_t rest = pm >> (p + 1); rest;) {
    const int gap = __ffs(rest);               // powers to the next one with a branch
    for (int k = 1; k < gap; ++k) {
      const float sc = scale_to(p + k);
#pragma unroll
      for (int i = 0; i < NP; ++i) advance(i, sc);
    }
    power(p, p + gap, std::false_type{});
    p += gap;
    rest >>= gap;
  }
  prefetch();                                  // in flight during the last products
  power(p, p, std::true_type{});
  const int ys = eb + e - kTapBits - kSampleBits;
  const uint32_t ny = d.n_y;
  const bool inside = wb + 512 * NT <= n;      // uniform: whole pairs, no bounds
  // the outputs against what may be missing of them
  const int left = inside ? 1 << 30 : n - (wb + 16 * NT * li + 2 * g);   // outputs from the lane's first on
  auto size = [&](int b) {                     // the lane's output b
    const int j = b >> 3, q = 2 * (b & 7);
    return 16 * j + 4 * ((b >> 1) & 3) + (b & 1) < left ? fmaxf(fabsf(tot[j][q]), fabsf(tot[j][q + 1])) : kHuge;
  };
  float least = kHuge, most = 0.f;
#pragma unroll
  for (int b = 0; b < 8 * NT; ++b) {
    least = fminf(least, size(b));
    most = fmaxf(most, size(b));
  }
  flags = 0;
  if (__any(least < thr || most < 8.f * thr)) {
    if (__any(most > 0.f && most < 8.f * thr)) return kPassLeft;
    int few = 0;
#pragma unroll
    for (int b = 0; b < 8 * NT; ++b) {
      const float m = size(b);
      const bool low = m > 0.f && m < thr;
      few += __popcll(__ballot(low));
      flags |= low ? 0x10000u << b : m == 0.f ? 1u << b : 0u;
    }
    if (few > kFew) return kPassLeft;
  }
  for (uint32_t k = 0; k < ny; ++k) {
    float2 *y = d.y[k] + wb + 16 * NT * li + 2 * g;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int o = 16 * j + 4 * q, p2 = wb + 16 * NT * li + 2 * g + o;
        const pair_u z = {ldexpf(tot[j][4 * q], ys), ldexpf(tot[j][4 * q + 1], ys),
                          ldexpf(tot[j][4 * q + 2], ys), ldexpf(tot[j][4 * q + 3], ys)};
        if (inside || p2 + 1 < n) st_pair(y + o, z);
        else if (p2 < n) st_global(y + o, make_float2(z.x, z.y));
      }
    }
  }
  return __any(flags != 0u) ? kPassCheck : kPassDone;
}
}  // namespace

// *ticket must be zero at launch (the producer of the item list clears it).
template <int TILE>
__global__ __launch_bounds__(256, 2) void k_fb_split(const FbFrameDesc *__restrict__ frames,
                                                     const WorkItem *__restrict__ items,
                                                     const uint32_t *__restrict__ n_items_ptr,
                                                     unsigned int *__restrict__ ticket) {
  constexpr int T = TILE, NTMAX = TILE >= 4096 ? 2 : 1, NPM = 4 * NTMAX + 1;
  constexpr int PL2 = 2 * split_plane(NTMAX) > 3 * kF32Plane ? 2 * split_plane(NTMAX) : 3 * kF32Plane;
  __shared__ SplitShared sh;
  __shared__ __align__(16) uint32_t s_plane[kSplitWaves][PL2];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t *plane = s_plane[w];
  const uint32_t n_items = *n_items_ptr;
  const bool tickets = 2ull * gridDim.x < n_items;
  // what the tap table holds: a bank's powers (tab_bank), or the sums of a
  // mask over several banks (tab_bank -1; every bit of the mask may be a branch)
  const float2 *tab_taps = nullptr;
  int tab_bank = -1;
  uint32_t tab_mask = 0, par = 0;
  pair_u v[NPM];
  auto pass_nt = [&](int left) { return NTMAX > 1 && left > 2048 ? 2 : 1; };
  CItem *const list = (CItem *)items;
  CDesc *const descs = (CDesc *)frames;
  // first window of an item
  auto item_window = [&](uint32_t i) -> const float2 * {
    if (i >= n_items) return nullptr;
    CDesc &d = descs[list[i].frame];
    if (d.route || !d.mask) return nullptr;
    const int n0 = (int)list[i].tile * T;
    return window_ptr<NTMAX>(d, n0, pass_nt((int)d.n - n0), w);
  };
  uint32_t it = blockIdx.x, it1 = blockIdx.x + gridDim.x;
  prefetch_window<NTMAX>(item_window(it), lane, v);
  while (it < n_items) {
    if (t == 0) sh.next[par] = tickets ? 2u * gridDim.x + atomicAdd(ticket, 1u) : n_items;
    CDesc &d = descs[list[it].frame];
    const int n0 = (int)list[it].tile * T;
    const int rem = min(T, (int)d.n - n0);
    const float2 *const next_item = item_window(it1);
    const uint32_t kfull = (1u << d.Kmax) - 1u;
    uint32_t pm = 0;
    int L = 1, nb = 0, bank1 = -1;
    for (uint32_t bank = 0; bank < d.n_banks; ++bank) {
      const uint32_t bm = (d.mask >> (bank * d.Kmax)) & kfull;
      pm |= bm;
      if (bm) { L = max(L, (int)d.L[bank]); ++nb; bank1 = (int)bank; }
    }
    if (nb > 1) bank1 = -1;
    if (d.route || !pm) {
      for (int k = t; k < rem; k += 256) {
        const float2 z = d.route ? ld_global(d.x + n0 + k) : make_float2(0.f, 0.f);
        for (uint32_t o = 0; o < d.n_y; ++o) st_global(d.y[o] + n0 + k, z);
      }
      prefetch_window<NTMAX>(next_item, lane, v);
    } else {
      const uint32_t tm = bank1 >= 0 ? 0u : d.mask;
      if (d.taps != tab_taps || bank1 != tab_bank || tm != tab_mask) {   // uniform across the workgroup
        tab_taps = d.taps;
        tab_bank = bank1;
        tab_mask = tm;
        if (L <= 33) build_table<6>(d, bank1, sh);
        else if (L <= 49) build_table<8>(d, bank1, sh);
        else build_table<10>(d, bank1, sh);
      }
      for (int off = 0; off < rem;) {
        const int nt = pass_nt(rem - off), step = 2048 * nt;
        const float2 *const next =
            off + step < rem ? window_ptr<NTMAX>(d, n0 + off + step, pass_nt(rem - off - step), w) : next_item;
        auto prefetch = [&]() { prefetch_window<NTMAX>(next, lane, v); };
        int end;
        uint32_t flags = 0;
#define PRUNE_SP(nt, s) \
  end = split_pass<(nt <= NTMAX ? nt : 1), s, NTMAX>(d, n0 + off, pm, sh, plane, v, lane, w, flags, prefetch)
        if (NTMAX > 1 && nt > 1) {
          if (L <= 33) PRUNE_SP(2, 6);
          else if (L <= 49) PRUNE_SP(2, 8);
          else PRUNE_SP(2, 10);
        } else {
          if (L <= 33) PRUNE_SP(1, 6);
          else if (L <= 49) PRUNE_SP(1, 8);
          else PRUNE_SP(1, 10);
        }
#undef PRUNE_SP
        if (end != kPassDone) {
          const int wb = n0 + off + w * 512 * nt;
          const bool two = NTMAX > 1 && nt > 1;
          const uint32_t zeros = flags & 0xffffu;
          if (end == kPassCheck) {
            __builtin_amdgcn_s_waitcnt(0);     // for the outputs that are written again
            asm volatile("" ::: "memory");
            if (__any(zeros != 0u) && !(two ? silent_windows<NTMAX>(d, wb, L, zeros, plane, lane)
                                            : silent_windows<1>(d, wb, L, zeros, plane, lane)))
              end = kPassLeft;
            else if (two) fix_outputs<NTMAX>(d, wb, flags >> 16, lane);
            else fix_outputs<1>(d, wb, flags >> 16, lane);
          }
          if (end == kPassLeft) {
            for (int o = 0; o < 512 * nt && wb + o < (int)d.n; o += 512)
              fp32_outputs(d, wb + o, (float *)plane, lane);
          }
          prefetch();                          // (again: the calls took its registers)
        }
        off += step;
      }
    }
    __syncthreads();
    it = it1;
    it1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.next[par]);
    par ^= 1u;
  }
}

template <int TILE>
void launch_fb_split(const FbFrameDesc *f, const WorkItem *it, const uint32_t *n,
                     unsigned int *ticket, uint32_t grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (e0 || e1)
    hipExtLaunchKernelGGL((k_fb_split<TILE>), dim3(grid), dim3(256), 0, s, e0, e1, 0, f, it, n, ticket);
  else
    hipLaunchKernelGGL((k_fb_split<TILE>), dim3(grid), dim3(256), 0, s, f, it, n, ticket);
}

template <int TILE>
int fb_split_resident() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(&k_fb_split<TILE>), 256, 0) !=
      hipSuccess)
    n = 0;
  return n;
}

#define PRUNE_SPLIT_INST(tile)                                                                             \
  template int fb_split_resident<tile>();                                                                  \
  template void launch_fb_split<tile>(const FbFrameDesc *, const WorkItem *, const uint32_t *,             \
                                    unsigned int *, uint32_t, hipStream_t, hipEvent_t, hipEvent_t);
PRUNE_SPLIT_INST(8192)
PRUNE_SPLIT_INST(4096)
PRUNE_SPLIT_INST(2048)
#undef PRUNE_SPLIT_INST

}  // namespace prune
