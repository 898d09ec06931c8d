// Filter-bank forward kernels (the fused basis-generation + FIR + branch-sum
// actor of the DPD application, Sec. VII-A; the DPG of poly, FIR_b and add
// merged into one firing as in the actor merging of Sec. VII-A's DNN case).
//
// For one firing with branch mask m over banks of Kmax branches:
//   y[n] = sum_{d in m} sum_{l < L_d} h_d[l] |x[n-l]|^{p_d} x[n-l],  p_d = d mod Kmax
// Within one bank all branches share L, so the branch sum is rewritten per
// (n, l) as a polynomial in r = |x[n-l]| evaluated by Horner's rule:
//   y[n] = sum_l x[n-l] * P_l(r[n-l]),  P_l(r) = sum_{b active} h_b[l] r^{b-1}
// which costs 2(KH-1)+4 fp32 FMAs per (n, l) instead of 4 KH (KH = highest
// active branch + 1 of the bank; inactive lower branches get zero
// coefficients).  The arithmetic is fp32 with FMA contraction; r is the
// correctly rounded sqrtf of fmaf(re, re, im^2) (magnitude).
//
// Data layout: frames are complex64 (float2) blocks in HBM.  A work item is
// one tile of T = J*WG consecutive outputs of one frame.  The tile's input
// window [n0 - (Lpad-1), n0 + T) is staged in LDS as three fp32 planes (re,
// im, r) with one pad element per J: lane t reads at stride J+1 words (9 or
// 5, odd, so the lanes of a read fall in distinct banks), and every window
// and coefficient read of a chunk is a constant offset from one base.  At
// 12 bytes per window sample the J = 8, 256-thread kernel needs 33.6 KB of
// LDS, so four workgroups fit on a CU, as many as its registers allow.
// Window positions before the frame come from the frame's halo (the stream's
// past samples), positions after the frame are zero.  Each lane computes J
// consecutive outputs from a register window of 2J-1 samples per chunk of J
// taps; the tap coefficients of the chunk are LDS broadcasts.
//
// What bounds it.  1024 frames x 65536, 2 to 10 branches, 10 taps: 355 us, from
// 433 (the samples alone take 230 us at the copy rate, the multiply-adds about
// 280 at their ceiling); one branch of 8 taps: 250 us, from 420.  What made
// the difference: tickets from eight counters instead of one (TileQueue), no
// window held in registers for the next tile (69 registers: seven workgroups
// of the J = 4 kernel share a CU and hide each other's loads), and outputs
// stored two at a time (365 to 355, and 286 to 250).
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>

#include "prune_internal.h"
#include "runtime_kernels.h"
#include "split_common.h"

namespace prune {

constexpr int kMaxKH = 10;

// Window layout: one pad element per J in each plane, so position t*J + k
// (k >= 0) is at t*(J+1) + k + k/J: a per-lane part plus a part uniform
// across lanes.  Lanes read words J+1 apart, an odd stride, so they hit
// distinct banks.
template <int J>
__device__ __forceinline__ int pidx(int i) { return i + i / J; }

// Coefficient table layout: tap-major, coef[l * kMaxKH + b], so the
// coefficients of a chunk are at constant offsets from one base.  Chunk c
// holds taps cJ .. cJ+J-1; the last one holds only L - (nchunks-1) J real
// taps (the rest are zero padding) and stops there.
template <int KH, int J, int G, bool PIPE>
__device__ __forceinline__ void horner_pass(const float *__restrict__ wre,
                                            const float *__restrict__ wim,
                                            const float *__restrict__ wrr,
                                            const float2 *__restrict__ coef, int Lpad, int L,
                                            int t, float *accr, float *acci) {
  const int nchunks = Lpad / J;
  for (int c = 0; c < nchunks; ++c) {
    // window positions t*J + k0 + w, k0 = Lpad - (c+1) J (a multiple of J)
    const int k0 = Lpad - c * J - J;
    const int wb = t * (J + 1) + k0 + k0 / J;   // this lane's part plus the chunk's
    const float2 *cb = coef + c * J * kMaxKH;
    float xr[2 * J - 1], xi[2 * J - 1], rr[2 * J - 1];
#pragma unroll
    for (int w = 0; w < 2 * J - 1; ++w) {
      const int q = wb + w + w / J;
      xr[w] = wre[q];
      xi[w] = wim[q];
      rr[w] = wrr[q];
    }
    // PIPE: the coefficients of tap i+1 are read from LDS while tap i
    // computes (every tap index below Lpad is in the table, zero-padded)
    float2 cn[KH];
    if (PIPE) {
#pragma unroll
      for (int b = 0; b < KH; ++b) cn[b] = cb[b];
    }
#pragma unroll
    for (int i = 0; i < J; ++i) {
      if (c * J + i >= L) break;   // uniform: zero-padded taps of the last chunk
      float2 cf[KH];
#pragma unroll
      for (int b = 0; b < KH; ++b) cf[b] = PIPE ? cn[b] : cb[i * kMaxKH + b];
      if (PIPE && i + 1 < J) {
#pragma unroll
        for (int b = 0; b < KH; ++b) cn[b] = cb[(i + 1) * kMaxKH + b];
      }
      // the Horner chains of G outputs advance together, one branch at a
      // time, so a wave has 2G independent FMAs in flight
#pragma unroll
      for (int j0 = 0; j0 < J; j0 += G) {
        float ar[G], ai[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          ar[g] = cf[KH - 1].x;
          ai[g] = cf[KH - 1].y;
        }
#pragma unroll
        for (int b = KH - 2; b >= 0; --b) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int w = j0 + g - i + J - 1;
            ar[g] = fmaf(ar[g], rr[w], cf[b].x);
            ai[g] = fmaf(ai[g], rr[w], cf[b].y);
          }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int j = j0 + g, w = j - i + J - 1;
          accr[j] = fmaf(xr[w], ar[g], accr[j]);
          accr[j] = fmaf(-xi[w], ai[g], accr[j]);
          acci[j] = fmaf(xr[w], ai[g], acci[j]);
          acci[j] = fmaf(xi[w], ar[g], acci[j]);
        }
      }
    }
  }
}

template <int J, int G, bool PIPE>
__device__ __forceinline__ void horner_dispatch(int KH, const float *wre, const float *wim,
                                                const float *wrr, const float2 *coef, int Lpad,
                                                int L, int t, float *accr, float *acci) {
#define PRUNE_HP(k) horner_pass<k, J, G, PIPE>(wre, wim, wrr, coef, Lpad, L, t, accr, acci)
  switch (KH) {
    case 0: break;
    case 1: PRUNE_HP(1); break;
    case 2: PRUNE_HP(2); break;
    case 3: PRUNE_HP(3); break;
    case 4: PRUNE_HP(4); break;
    case 5: PRUNE_HP(5); break;
    case 6: PRUNE_HP(6); break;
    case 7: PRUNE_HP(7); break;
    case 8: PRUNE_HP(8); break;
    case 9: PRUNE_HP(9); break;
    default: PRUNE_HP(10); break;
  }
#undef PRUNE_HP
}

// A tile's operands: the frame's samples, the stream before it, and its taps.
struct TileIn {
  const float2 *x;      // sample 0 of the frame
  const float2 *past;   // past[p] is sample p < 0
  const float2 *taps;   // [n_banks][Kmax][Lmax]
  int n, before;        // samples of the frame, and of the stream before it that exist
  uint32_t mask, route, n_banks, Kmax, Lmax;
};

template <int J, int WG>
struct TileShared {
  static constexpr int WMAX = J * WG + PRUNE_MAX_L - 1;   // window of a tile
  static constexpr int WP = WMAX + WMAX / J + 1;          // with the pads
  float wre[WP], wim[WP], wrr[WP];
  float2 coef[kMaxKH * PRUNE_MAX_L];
};

// The J outputs of this thread from n0 + t J on.  bank_L(b): taps of bank b.
// All of a bank's loads are issued before the first is used.
template <int J, int WG, int G, bool PIPE, class BankL>
__device__ __forceinline__ void fb_tile(const TileIn &in, int n0, const BankL &bank_L, TileShared<J, WG> &sh, int t,
                                        float (&accr)[J], float (&acci)[J]) {
  constexpr int T = J * WG, NIT = (TileShared<J, WG>::WMAX + WG - 1) / WG;
  constexpr int NC = (kMaxKH * PRUNE_MAX_L + WG - 1) / WG;
#pragma unroll
  for (int j = 0; j < J; ++j) accr[j] = acci[j] = 0.f;
  if (in.route) {   // passthrough-routed frame: y = x
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int p = n0 + t * J + j;
      if (p < in.n) {
        const float2 v = ld_global(in.x + p);
        accr[j] = v.x;
        acci[j] = v.y;
      }
    }
    return;
  }
  const uint32_t kfull = (1u << in.Kmax) - 1u;
  bool later = false;
  for (uint32_t bank = 0; bank < in.n_banks; ++bank) {
    const uint32_t bmask = (in.mask >> (bank * in.Kmax)) & kfull;
    if (!bmask) continue;
    const int KH = 32 - __clz(bmask), L = (int)bank_L(bank), Lpad = (L + J - 1) / J * J, WN = T + Lpad - 1;
    const float2 *tb = in.taps + (size_t)bank * in.Kmax * in.Lmax;
    float2 v[NIT], c[NC];
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int k = t + i * WG, p = n0 - (Lpad - 1) + k;
      v[i] = make_float2(0.f, 0.f);
      if (k < WN && p < in.n && p >= -in.before) v[i] = ld_global((p >= 0 ? in.x : in.past) + p);
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = t + i * WG, b = k / Lpad, l = k - b * Lpad;
      c[i] = make_float2(0.f, 0.f);
      if (k < KH * Lpad && ((bmask >> b) & 1u) && l < L) c[i] = ld_global(tb + (size_t)b * in.Lmax + l);
    }
    if (later) __syncthreads();   // readers of the bank before
    later = true;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int k = t + i * WG;
      if (k < WN) {
        const int q = pidx<J>(k);
        sh.wre[q] = v[i].x;
        sh.wim[q] = v[i].y;
        sh.wrr[q] = magnitude(v[i].x, v[i].y);
      }
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = t + i * WG, b = k / Lpad, l = k - b * Lpad;
      if (k < KH * Lpad) sh.coef[l * kMaxKH + b] = c[i];
    }
    __syncthreads();
    // a wave whose outputs all lie beyond the frame's end (the last tile of a
    // frame) stores nothing and skips the arithmetic (KH 0); the condition is
    // uniform across the wave
    horner_dispatch<J, G, PIPE>(n0 + (t & ~63) * J < in.n ? KH : 0, sh.wre, sh.wim, sh.wrr, sh.coef, Lpad, L, t, accr,
                                acci);
  }
}

// Outputs p .. p + J - 1 of a frame of n samples, two to a store.
template <int J>
__device__ __forceinline__ void store_outputs(float2 *y, int p, int n, const float (&accr)[J], const float (&acci)[J]) {
#pragma unroll
  for (int j = 0; j + 1 < J; j += 2) {
    if (p + j + 1 < n) st_pair(y + p + j, pair_u{accr[j], acci[j], accr[j + 1], acci[j + 1]});
    else if (p + j < n) st_global(y + p + j, make_float2(accr[j], acci[j]));
  }
  if (J & 1)
    if (p + J - 1 < n) st_global(y + p + J - 1, make_float2(accr[J - 1], acci[J - 1]));
}

// Persistent form over a work list (TileQueue).  Thread 0 takes the ticket of
// the tile after next at the start of a tile, so that its round trip overlaps
// a whole tile.
template <int J, int WG, int WAVES, int G, bool PIPE>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_fb_forward(const FbFrameDesc *__restrict__ frames, const WorkItem *__restrict__ items,
                  const uint32_t *__restrict__ n_items_ptr, unsigned int *__restrict__ ticket) {
  typedef const __attribute__((address_space(4))) FbFrameDesc CDesc;
  typedef const __attribute__((address_space(4))) WorkItem CItem;
  __shared__ TileShared<J, WG> sh;
  __shared__ uint32_t s_next[2];
  const int t = threadIdx.x;
  const uint32_t n_items = *n_items_ptr;
  const TileQueue tq(n_items, ticket);
  uint32_t k = tq.first(), k1 = tq.second(), par = 0;
  while (k < tq.count) {
    const uint32_t it = tq.item(k);
    if (t == 0) s_next[par] = tq.later();
    CDesc &d = ((CDesc *)frames)[((CItem *)items)[it].frame];
    const int n0 = (int)((CItem *)items)[it].tile * (J * WG);
    TileIn in;
    in.x = d.x; in.past = d.halo + ((int)d.Lmax - 1); in.taps = d.taps;
    in.n = (int)d.n; in.before = (int)d.halo_valid;
    in.mask = d.mask; in.route = d.route; in.n_banks = d.n_banks; in.Kmax = d.Kmax; in.Lmax = d.Lmax;
    float accr[J], acci[J];
    fb_tile<J, WG, G, PIPE>(in, n0, [&](uint32_t b) { return d.L[b]; }, sh, t, accr, acci);
    for (uint32_t o = 0; o < d.n_y; ++o) {
      store_outputs<J>(d.y[o], n0 + t * J, in.n, accr, acci);
    }
    __syncthreads();   // the tile's readers are done; s_next is written
    k = k1;
    k1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_next[par]);
    par ^= 1u;
  }
}

// One launch for short work: a workgroup per tile, (frame, tile) from its
// index, everything else from the frame's own record, so that nothing has to
// be prepared.  Grid: n_frames times the tiles of the longest frame;
// workgroups beyond their frame's end leave at once.
template <int J, int WG>
__global__ __launch_bounds__(WG) void k_fb_small(prune_fb_desc d, const float2 *__restrict__ xs,
                                                 const float2 *__restrict__ taps,
                                                 const prune_fb_frame *__restrict__ frames, float2 *__restrict__ ys,
                                                 uint32_t per) {
  constexpr int T = J * WG;
  __shared__ TileShared<J, WG> sh;
  typedef const __attribute__((address_space(4))) prune_fb_frame cframe;
  const uint32_t f = blockIdx.x / per;
  cframe &fr = ((cframe *)frames)[f];
  const uint32_t t0 = fr.t0, stream = fr.stream;
  const int t = threadIdx.x, n = (int)fr.n, n0 = (int)(blockIdx.x - f * per) * T;
  if (n0 >= n || stream >= d.n_streams || (uint64_t)t0 + (uint32_t)n > d.stream_len || (uint32_t)n > d.max_frame_len)
    return;
  uint32_t Lmax = 1;
  for (uint32_t b = 0; b < d.n_banks; ++b) Lmax = max(Lmax, d.L[b]);
  TileIn in;
  in.x = in.past = xs + (size_t)stream * d.stream_len + t0;
  in.taps = taps + (size_t)stream * d.n_banks * d.Kmax * Lmax;
  in.n = n; in.before = (int)min(t0, Lmax - 1);
  in.mask = fr.mask; in.route = fr.route; in.n_banks = d.n_banks; in.Kmax = d.Kmax; in.Lmax = Lmax;
  float accr[J], acci[J];
  fb_tile<J, WG, J, false>(in, n0, [&](uint32_t b) { return d.L[b]; }, sh, t, accr, acci);
  store_outputs<J>(ys + (size_t)stream * d.stream_len + t0, n0 + t * J, n, accr, acci);
}

// ---------------------------------------------------------------- variants
struct FbVariant {
  const char *name;
  int tile, WG;   // outputs per work item, threads per workgroup
  void (*launch)(const FbFrameDesc *, const WorkItem *, const uint32_t *, unsigned int *,
                 uint32_t grid, hipStream_t, hipEvent_t, hipEvent_t);
  int (*resident)();   // workgroups of the kernel resident per CU
};

template <int J, int WG, int WAVES, int G = J, bool PIPE = false>
static int fwd_resident() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(&k_fb_forward<J, WG, WAVES, G, PIPE>),
                                                   WG, 0) != hipSuccess)
    n = 0;
  return n;
}

// With events, the dispatch itself records the kernel's start and end
// (hipExtLaunchKernelGGL): no marker packets, no gaps around the kernel.
template <int J, int WG, int WAVES, int G = J, bool PIPE = false>
static void launch_fwd(const FbFrameDesc *f, const WorkItem *it, const uint32_t *n,
                       unsigned int *ticket, uint32_t grid, hipStream_t s, hipEvent_t e0,
                       hipEvent_t e1) {
  if (e0 || e1)
    hipExtLaunchKernelGGL((k_fb_forward<J, WG, WAVES, G, PIPE>), dim3(grid), dim3(WG), 0, s, e0, e1, 0, f, it, n, ticket);
  else
    hipLaunchKernelGGL((k_fb_forward<J, WG, WAVES, G, PIPE>), dim3(grid), dim3(WG), 0, s, f, it, n, ticket);
}

static const FbVariant kVariants[] = {
    // vector Horner kernels: J outputs per lane, WG threads, waves-per-EU
    // hint, Horner chains of G outputs advanced together, next tap's
    // coefficients read ahead (p) or not (w)
    {"valu_horner_J8_WG256_p4", 8 * 256, 256, launch_fwd<8, 256, 1, 4, true>, fwd_resident<8, 256, 1, 4, true>},
    {"valu_horner_J4_WG256_w3", 4 * 256, 256, launch_fwd<4, 256, 3>, fwd_resident<4, 256, 3>},
    {"valu_horner_J8_WG128_w2", 8 * 128, 128, launch_fwd<8, 128, 2>, fwd_resident<8, 128, 2>},
    {"valu_horner_J4_WG128_w4", 4 * 128, 128, launch_fwd<4, 128, 4>, fwd_resident<4, 128, 4>},
    {"valu_horner_J8_WG256_p2", 8 * 256, 256, launch_fwd<8, 256, 1, 2, true>, fwd_resident<8, 256, 1, 2, true>},
    // split half-precision matrix-core kernels (fb_split.hip) by tile
    {"mfma_split_f16_T8192", 8192, 256, launch_fb_split<8192>, fb_split_resident<8192>},
    {"mfma_split_f16_T4096", 4096, 256, launch_fb_split<4096>, fb_split_resident<4096>},
    {"mfma_split_f16_T2048", 2048, 256, launch_fb_split<2048>, fb_split_resident<2048>},
};

constexpr int kNumVector = 5;   // the vector kernels come first

int fb_variant_count() { return (int)(sizeof(kVariants) / sizeof(kVariants[0])); }
const char *fb_variant_name(int v) {
  return (v >= 1 && v <= fb_variant_count()) ? kVariants[v - 1].name : "auto";
}
int fb_variant_tile(int v) { return kVariants[v - 1].tile; }
int fb_variant_wg(int v) { return kVariants[v - 1].WG; }
bool fb_variant_allowed(int v, uint32_t min_taps) {
  return v <= kNumVector || min_taps >= kSplitMinTaps;
}

// Queried once per variant (on the current device; every device here is
// the same gfx950 part).
int fb_variant_resident(int v) {
  static std::atomic<int> cache[sizeof(kVariants) / sizeof(kVariants[0])] = {};
  int n = cache[v - 1].load();
  if (n <= 0) {
    n = std::max(1, kVariants[v - 1].resident());
    cache[v - 1].store(n);
  }
  return n;
}

void fb_forward_launch(int v, const FbFrameDesc *frames, const WorkItem *items,
                       const uint32_t *n_items, unsigned int *ticket, uint32_t grid,
                       hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  kVariants[v - 1].launch(frames, items, n_items, ticket, grid, s, e0, e1);
}

template <int J>
static void launch_small(const prune_fb_desc &d, const float2 *x, const float2 *taps, const prune_fb_frame *frames,
                         float2 *y, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const uint32_t per = std::max<uint32_t>(1, (d.max_frame_len + 256 * J - 1) / (256 * J));
  const dim3 grid(d.n_frames * per);
  if (e0 || e1)
    hipExtLaunchKernelGGL((k_fb_small<J, 256>), grid, dim3(256), 0, s, e0, e1, 0, d, x, taps, frames, y, per);
  else
    hipLaunchKernelGGL((k_fb_small<J, 256>), grid, dim3(256), 0, s, d, x, taps, frames, y, per);
}

// Outputs a lane computes in the one-launch form, or 0 for the work lists.
// n outputs of whole frames, K = 10, L = 10 (kernel alone, J = 1, 2, 4): 1000:
// 4.0, 4.3, 5.2 us; 16384: 4.7, 5.0, 6.1; 262144: 6.8, 6.2, 7.0; 524288: 11.7,
// 9.4, 9.1; so the most that leaves two workgroups a CU.  With the list's
// preparation, which walks the frames in one workgroup, the work lists take 12
// us where this takes 7 (up to 65536 outputs; 7 is the launch itself), 29.6
// against 21.9 at 2M, 135 against 111 at 16M, and win from about 50M on (373
// against 434 at 67M).  With the split kernel's tap counts they win earlier:
// 21.0 against 11.9 us at 524288 (26 taps), 27.4 against 31.1 at 1M (64).
// A workgroup beyond its frame's end costs 1.4 ns (2000 frames of 300, up to
// 65536 allowed: 190 us against 42), hence the bound on the grid.
int fb_small_outputs(const prune_fb_desc &d) {
  const uint64_t outputs = (uint64_t)d.n_frames * d.max_frame_len;
  const uint32_t shortest = *std::min_element(d.L, d.L + d.n_banks);
  if (outputs > (shortest < kSplitMinTaps ? 1u << 24 : 1u << 19)) return 0;
  const int J = outputs >= 1u << 19 ? 4 : outputs >= 1u << 18 ? 2 : 1;
  const uint64_t grid = (uint64_t)d.n_frames * ((d.max_frame_len + 256 * J - 1) / (256 * J));
  const uint64_t tiles = (uint64_t)d.n_streams * d.stream_len / (256 * J) + d.n_frames;   // at most
  return grid <= std::min<uint64_t>(2 * tiles + 4096, 1u << 23) ? J : 0;   // below 2^32 threads
}

void fb_small_launch(const prune_fb_desc &d, const float2 *x, const float2 *taps, const prune_fb_frame *frames,
                     float2 *y, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (fb_small_outputs(d)) {
    case 1: launch_small<1>(d, x, taps, frames, y, s, e0, e1); break;
    case 2: launch_small<2>(d, x, taps, frames, y, s, e0, e1); break;
    default: launch_small<4>(d, x, taps, frames, y, s, e0, e1); break;
  }
}

}  // namespace prune
