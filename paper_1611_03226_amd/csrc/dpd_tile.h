// One tile of predistortion outputs inside one firing (device code shared by
// the single-actor batch kernel and the multi-instance persistent kernel).
//
// Inside a firing every active branch reads the same input samples, so the
// branch sum is evaluated per tap as a polynomial in p = |x|^2 (Horner over
// branches, Sec. 4.2 actor body):
//   y[t] = sum_m x[t-m] * P_m(p[t-m]),   P_m(p) = sum_{b<B} h[b][m] p^b.
// With a branch set that is not a prefix, the coefficients of the inactive
// branches below the highest active one enter the polynomial as zeros.
// The samples before the firing start are staged as zeros; the taps that
// reach there read branch b's own history and are added per branch.
#pragma once

#include "common.h"

namespace dfh {

// Read-only device data seen through the constant address space: loads from
// it at wavefront-uniform addresses become scalar loads into SGPRs, which the
// FMAs read directly (no VGPRs, no LDS traffic for the coefficients).  Only
// memory that no kernel of the launch writes may be read this way.
typedef const __attribute__((address_space(4))) float2 *cfloat2p;

template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_const(const T *p) {
  return (const __attribute__((address_space(4))) T *)p;
}

// Element i of a constant-space complex array.
__device__ __forceinline__ float2 ldc(cfloat2p p, int i) {
  const __attribute__((address_space(4))) float *f = (const __attribute__((address_space(4))) float *)p;
  return make_float2(f[2 * i], f[2 * i + 1]);
}

// Element i, or +0 when `keep` is clear (all-ones / all-zero word: the
// select is a bitwise AND on the uniform coefficient words).
__device__ __forceinline__ float2 ldc_masked(cfloat2p p, int i, uint32_t keep) {
  const float2 v = ldc(p, i);
  return make_float2(__builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v.x) & keep),
                     __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v.y) & keep));
}

// LDS slot of window sample i for K outputs per thread: one pad slot per K
// samples, so a wavefront's K-strided 8-byte window reads start 2K + 2 words
// apart and each half wavefront covers the 64 banks once (K = 4 with one pad
// per 8 samples put two lanes on a bank).  Samples K apart are K + 1 slots
// apart, so a thread's reads of sample K * thread + c are one base and an
// offset known at compile time.
template <int K>
__host__ __device__ constexpr int lds_slot(int i) { return (int)((unsigned)i + (unsigned)i / K); }
template <int K>
__host__ __device__ constexpr int lds_window(int n) { return lds_slot<K>(n) + 1; }

// Coefficients as the bodies read them: [taps][kCoefRow] complex, tap-major,
// with a fixed row length, so that the branches of one tap are consecutive
// (a few wide scalar loads instead of one per branch) at offsets known at
// compile time.

// Taps of K consecutive outputs q0..q0+K-1.  Tap m of output q0+k reads
// window sample k+M-1-m, so iterating the taps in order slides a window of
// K samples (one new LDS read per tap; the shift is a register rename).
// Reads stay inside the window buffer (index < tile+M-1); in a partial tile,
// slots past the staged samples only feed outputs that are not stored.
// ht: the firing's coefficients, tap-major (uniform address: scalar loads).
// MASKED: set is the firing's branch set (B = its Horner length) and the
// coefficients of branches outside it read as zero; without MASKED the set
// is the prefix 0..B-1 and the coefficients are used as loaded.
// Software pipeline of depth one: tap m+1's coefficients and sample are
// loaded before tap m's arithmetic (tap_fence).
// MT: the tap count when it is compiled in (4, 8, 16), else 0 and the taps
// are a loop over Mr, K taps a turn (the window's register rename repeats
// after K taps), and the remaining ones under uniform branches.
template <int K, int B, bool MASKED>
__device__ __forceinline__ void load_coefs(cfloat2p row, uint32_t set, float2 (&hc)[B]) {
#pragma unroll
  for (int b = 0; b < B; ++b) {
    if constexpr (MASKED) hc[b] = ldc_masked(row, b, 0u - ((set >> b) & 1u));
    else hc[b] = ldc(row, b);
  }
}

// One tap for the K outputs: y[k] += x P(p).
template <int K, int B>
__device__ __forceinline__ void horner_tap(const float2 (&hc)[B], const float2 (&wv)[K], const float (&pv)[K],
                                           float (&ar)[K], float (&ai)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float Pr = hc[B - 1].x, Pi = hc[B - 1].y;
#pragma unroll
    for (int b = B - 2; b >= 0; --b) {
      Pr = fmaf(Pr, pv[k], hc[b].x);
      Pi = fmaf(Pi, pv[k], hc[b].y);
    }
    ar[k] = fmaf(wv[k].x, Pr, ar[k]);
    ar[k] = fmaf(-wv[k].y, Pi, ar[k]);
    ai[k] = fmaf(wv[k].x, Pi, ai[k]);
    ai[k] = fmaf(wv[k].y, Pr, ai[k]);
  }
}

// Nothing is scheduled across: a tap's loads, its arithmetic and the first
// use of what was loaded stay in that order, so the one wait of a tap (LDS
// and scalar loads return out of order, it is for all of them) comes after
// the whole arithmetic and before the next loads.  Left to itself the
// scheduler moves the loads down to their use.
__device__ __forceinline__ void tap_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The window moved by one sample.
template <int K>
__device__ __forceinline__ void slide(float2 (&wv)[K], float (&pv)[K], float2 wn) {
#pragma unroll
  for (int k = K - 1; k > 0; --k) {
    wv[k] = wv[k - 1];
    pv[k] = pv[k - 1];
  }
  wv[0] = wn;
  pv[0] = fmaf(wn.x, wn.x, wn.y * wn.y);   // explicit: no contraction freedom
}

// One tap with the next tap's loads in flight: coefficients from `next`, the
// sample that enters the window from `in()`.
template <int K, int B, bool MASKED, class In>
__device__ __forceinline__ void piped_tap(cfloat2p next, uint32_t set, In in, float2 (&hc)[B], float2 (&wv)[K],
                                          float (&pv)[K], float (&ar)[K], float (&ai)[K]) {
  float2 hn[B];
  load_coefs<K, B, MASKED>(next, set, hn);
  const float2 wn = in();
  tap_fence();
  horner_tap<K, B>(hc, wv, pv, ar, ai);
  tap_fence();
  slide<K>(wv, pv, wn);
#pragma unroll
  for (int b = 0; b < B; ++b) hc[b] = hn[b];
  tap_fence();
}

template <int MT, int K, int B, bool MASKED>
__device__ __forceinline__ void horner_taps(cfloat2p ht, uint32_t set, const float2 *sx, int q0, int Mr,
                                            float (&ar)[K], float (&ai)[K]) {
  float2 wv[K];
  float pv[K];
  float2 hc[B];
  const int M = MT ? MT : Mr;
  const float2 *wp = sx + q0 / K * (K + 1);              // sample q0, q0 a multiple of K
#pragma unroll
  for (int k = 0; k < K; ++k) {
    wv[k] = wp[lds_slot<K>(M - 1 + k)];
    pv[k] = fmaf(wv[k].x, wv[k].x, wv[k].y * wv[k].y);
  }
  load_coefs<K, B, MASKED>(ht, set, hc);
  if constexpr (MT != 0) {
#pragma unroll
    for (int m = 0; m + 1 < MT; ++m)
      piped_tap<K, B, MASKED>(ht + (m + 1) * kCoefRow, set, [&] { return wp[lds_slot<K>(MT - 2 - m)]; }, hc, wv, pv, ar, ai);
    horner_tap<K, B>(hc, wv, pv, ar, ai);
  } else {
    int left = M - 1;                                    // taps after the current one
    for (; left >= K; left -= K) {
#pragma unroll
      for (int j = 0; j < K; ++j)
        piped_tap<K, B, MASKED>(ht + (j + 1) * kCoefRow, set, [&] { return wp[lds_slot<K>(left - 1 - j)]; }, hc, wv,
                                pv, ar, ai);
      ht += K * kCoefRow;
    }
#pragma unroll
    for (int j = 0; j < K - 1; ++j)
      if (left > j)                                      // uniform
        piped_tap<K, B, MASKED>(ht + (j + 1) * kCoefRow, set, [&] { return wp[lds_slot<K>(left - 1 - j)]; }, hc, wv,
                                pv, ar, ai);
    horner_tap<K, B>(hc, wv, pv, ar, ai);
  }
}

// LDS float2 slots for a firing's head corrections (M-1 outputs).
__host__ __device__ constexpr int lds_corr(int M) { return M > 1 ? M - 1 : 1; }

// Lane i of a 16-lane row receives lane i+S of the same row (0 past the
// row end): one DPP move.
template <int S>
__device__ __forceinline__ float row_shl(float v) {
  if constexpr (S == 0) {
    return v;
  } else {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x100 + S, 0xF, 0xF, true));
  }
}

// Taps m..M-1 of one branch's head correction for output i of the lane's
// row: psi of history sample i - m sits in lane (M-1) + i - m of the row.
// For m <= i (no history term) that lane is an idle lane of the row (psi 0)
// or past the row end (the shift yields 0), so every tap is summed.
template <int M, int m>
__device__ __forceinline__ void head_taps(cfloat2p hg, int b, float psr, float psi, float &sr, float &si) {
  const float2 c = ldc(hg, b * M + m);
  const float vr = row_shl<M - 1 - m>(psr), vi = row_shl<M - 1 - m>(psi);
  sr = fmaf(c.x, vr, sr);
  sr = fmaf(-c.y, vi, sr);
  si = fmaf(c.x, vi, si);
  si = fmaf(c.y, vr, si);
  if constexpr (m + 1 < M) head_taps<M, m + 1>(hg, b, psr, psi, sr, si);
}

// The same with the lane's branch's own coefficients (LDS or memory, hb[m]).
template <int M, int m>
__device__ __forceinline__ void row_taps(const float2 *hb, float psr, float psi, float &sr, float &si) {
  if constexpr (m < M) {
    const float2 c = hb[m];
    const float vr = row_shl<M - 1 - m>(psr), vi = row_shl<M - 1 - m>(psi);
    sr = fmaf(c.x, vr, sr);
    sr = fmaf(-c.y, vi, sr);
    si = fmaf(c.x, vi, si);
    si = fmaf(c.y, vr, si);
    row_taps<M, m + 1>(hb, psr, psi, sr, si);
  }
}

// Head corrections of up to four firings of one actor (one wavefront; lane
// 16*row + i serves firing `row`, history sample / output i).  Outputs
// q < M-1 of a firing reach back before its first sample, where branch b
// reads its own history source (the tail of its last feeding firing, or the
// carried state).  The tile body stages zeros there; this adds the
// difference:
//   corr[q] = sum_{b<B} sum_{m=q+1}^{M-1} h_b[m] psi_b(src_b[q-m]),
// accumulated branch by branch.  All history loads are issued at once; psi
// values move inside a row by DPP row shifts; the coefficients are the same
// for every row (uniform scalar loads).
//   B_of(row) -> branch set of the row's firing (empty: no correction)
//   src_of(row, b) -> history source firing of branch b (-1: carried state)
//   sample(row, b, pf, i) -> sample i of branch b's history
// Only branches b_first, b_first + b_step, ... are evaluated (a head pass may
// split a firing's branches over several wavefronts); for each, in
// increasing b, emit(b, active, sr, si) receives the lane's sum over that
// branch's taps (active: b is in the row's branch set).  The correction of
// (row, output i) is the sum of the active branches' values in increasing
// b, starting from 0 (every caller keeps that order, so all head passes
// round alike); it is meaningful where head_live() holds.
template <int M, int ROWS>
__device__ __forceinline__ bool head_live(uint32_t set) {
  const int lane = threadIdx.x & 63, row = lane >> 4, i = lane & 15;
  return row < ROWS && i < M - 1 && set != 0u;
}

template <int M, int ROWS, class BOf, class SrcOf, class Sample, class Emit>
__device__ __forceinline__ void head_correction(cfloat2p hg, BOf B_of, SrcOf src_of, Sample sample, int b_first,
                                                int b_step, Emit emit) {
  constexpr int L = M - 1;
  static_assert(L < 16, "one row of 16 lanes per firing");
  const int lane = threadIdx.x & 63, row = lane >> 4, i = lane & 15;
  const bool live = row < ROWS && i < L;
  const uint32_t all = row < ROWS ? (uint32_t)B_of(row) : 0u;
  uint32_t pick = 0u;                                  // branches of this pass
  for (int b = b_first; b < kMaxBranches; b += b_step) pick |= 1u << b;
  const uint32_t set = all & pick;
  const int B = set_len(set);
  int Bw = B;                                          // largest Horner length of the wavefront
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) Bw = max(Bw, __shfl_xor(Bw, o));
  Bw = __builtin_amdgcn_readfirstlane(Bw);
  int64_t pf[kMaxBranches];
#pragma unroll
  for (int b = 0; b < kMaxBranches; ++b) pf[b] = (in_set(set, b) && live) ? src_of(row, b) : -1;
  float2 xs[kMaxBranches];
#pragma unroll
  for (int b = 0; b < kMaxBranches; ++b)
    xs[b] = (in_set(set, b) && live) ? sample(row, b, pf[b], i) : make_float2(0.f, 0.f);
#pragma unroll
  for (int b = 0; b < kMaxBranches; ++b) {
    if (b >= Bw || !in_set(pick, b)) continue;         // uniform
    const float pp = fmaf(xs[b].x, xs[b].x, xs[b].y * xs[b].y);
    float pb = 1.f;
    for (int e = 0; e < b; ++e) pb *= pp;
    float sr = 0.f, si = 0.f;
    head_taps<M, 1>(hg, b, pb * xs[b].x, pb * xs[b].y, sr, si);
    emit(b, in_set(set, b), sr, si);
  }
}

// The same for any tap count (M <= RL + 1): rows of RL lanes, the taps a loop
// and psi moved by lane shuffles; branches b_first, b_first + 4, ...
// (src_of also takes which of them it is).
template <int RL, class BOf, class SrcOf, class Sample, class Emit>
__device__ __forceinline__ void head_correction_any(cfloat2p hg, int M, BOf B_of, SrcOf src_of, Sample sample,
                                                    int b_first, Emit emit) {
  const int L = M - 1;
  const int lane = threadIdx.x & 63, row = lane / RL, i = lane % RL;
  const uint32_t set = (uint32_t)B_of(row);
  int Bw = set_len(set);                                 // largest Horner length of the wavefront
#pragma unroll
  for (int o = RL; o < 64; o <<= 1) Bw = max(Bw, __shfl_xor(Bw, o));
  Bw = __builtin_amdgcn_readfirstlane(Bw);
#pragma unroll
  for (int c = 0; c < kMaxBranches; c += 4) {
    const int b = c + b_first;
    if (b >= Bw) break;                                  // uniform
    float2 xv = make_float2(0.f, 0.f);
    if (in_set(set, b) && i < L) xv = sample(row, b, src_of(row, b, c / 4), i);
    const float pp = fmaf(xv.x, xv.x, xv.y * xv.y);
    float pb = 1.f;
    for (int e = 0; e < b; ++e) pb *= pp;
    const float pr = pb * xv.x, pi = pb * xv.y;
    float sr = 0.f, si = 0.f;
    for (int m = 1; m < M; ++m) {
      const float2 h = ldc(hg, b * M + m);
      const int from = RL * row + ((L + i - m) & (RL - 1));   // history sample i - m (meaningful for m > i)
      const float vr = __shfl(pr, from), vi = __shfl(pi, from);
      if (m > i) {
        sr = fmaf(h.x, vr, sr);
        sr = fmaf(-h.y, vi, sr);
        si = fmaf(h.x, vi, si);
        si = fmaf(h.y, vr, si);
      }
    }
    emit(b, in_set(set, b), sr, si);
  }
}

// The tile pipeline.  A workgroup of NT threads computes tiles of K*NT
// consecutive outputs of one firing (B uniform over the tile), walking the
// batch's tiles with a grid stride.  Loads are issued well before their use:
// the descriptor of tile i+2 and the window
// and head corrections of tile i+1 are loaded while tile i is computed.
// Bound by VALU issue (16 taps, 2^24 samples, mean length 5.5: 55 M wavefront
// instructions of arithmetic, 90 us of the chip's issue); the body takes
// 108 us there, 122 us before the taps were fenced (loads ahead of a tap, one
// wait behind it), the stores moved behind the wait for the next window, the
// window slots spread over all banks and the addresses made uniform bases
// with 32-bit offsets.  The run-time tap loop takes 22 us for 2^21 samples of
// 10 taps (mean length 6); one thread per sample and tap took 110 us.
// Samples before the firing start are staged as zeros; a firing's first
// M-1 outputs then add their head correction.  Every rounding step is an
// explicit fmaf or a single operation, so all kernels built from these
// pieces produce bit-identical outputs.

// Everything about one tile, uniform across the workgroup.
struct Job {
  const float2 *x;        // input ring
  float2 *y;              // output ring
  const float2 *h;        // coefficients of the firing's actor, tap-major [M][kCoefRow]
  const float2 *corr;     // the firing's head corrections [M-1] (used when head)
  int64_t x_mask, y_mask;
  int64_t xb, yb;         // ring positions of the tile's first input / output sample
  int nout;               // outputs in the tile
  uint32_t set;           // active branches of the firing (bit set)
  int B;                  // its Horner length (highest active branch + 1)
  int first;              // first tile of its firing (0/1): no samples before it
  int head;               // ... whose outputs take head corrections (0/1)
  int g;                  // firing (workgroups that form their own head corrections)
};

// Where a run of n consecutive ring samples from position p starts, and
// whether it runs past the ring's end (uniform; a linear array never does).
__device__ __forceinline__ bool ring_run(int64_t p, int64_t mask, int n, int64_t *slot) {
  *slot = p & mask;
  return mask >= 0 && *slot + n > mask + 1;
}

template <int K>
struct TileRegs {
  float2 win[K + 1];
  float2 cv;              // head correction of output threadIdx.x (< M-1)
};

// Loads of tile j into registers (issued early, consumed by commit): sample
// i of the window (i < nout + M - 1, the first M - 1 before the tile) by
// thread i mod NT.  Addresses are a uniform base and a 32-bit offset; a tile
// that runs past the ring's end (one in ring / tile) takes the masked form.
// Indices are clamped into the window, and below a firing's start onto its
// first sample (commit_tile writes 0 there), so that no load is conditional
// and none is waited for here.
// CORR: head corrections come from memory (else the workgroup forms them).
template <int K, bool CORR = true>
__device__ __forceinline__ void load_tile(TileRegs<K> &r, const Job &j, int M) {
  const int tid = threadIdx.x, nt = blockDim.x, lo = j.first ? M - 1 : 0, hi = j.nout + M - 2;
  int64_t slot;
  if (!ring_run(j.xb - (M - 1), j.x_mask, j.nout + M - 1, &slot)) {
    const char *p = (const char *)(j.x + slot);
#pragma unroll
    for (int u = 0; u < K; ++u)
      r.win[u] = *(const float2 *)(p + (uint32_t)min(max(tid + u * nt, lo), hi) * 8u);
    if (tid < M - 1) r.win[K] = *(const float2 *)(p + (uint32_t)min(K * nt + tid, hi) * 8u);
  } else {
#pragma unroll
    for (int u = 0; u < K; ++u) r.win[u] = j.x[(slot + min(max(tid + u * nt, lo), hi)) & j.x_mask];
    if (tid < M - 1) r.win[K] = j.x[(slot + min(K * nt + tid, hi)) & j.x_mask];
  }
  if (CORR && j.head && tid < M - 1) r.cv = j.corr[tid];
}

// Waits for the loads of load_tile.  The workgroup does so before it stores a
// tile's outputs: loads and stores count on one counter in issue order, and a
// wait at the next commit would be for the stores too.
template <int K, bool CORR = true>
__device__ __forceinline__ void settle(TileRegs<K> &r) {
#pragma unroll
  for (int u = 0; u < K + 1; ++u) asm volatile("" : "+v"(r.win[u].x), "+v"(r.win[u].y));
  if (CORR) asm volatile("" : "+v"(r.cv.x), "+v"(r.cv.y));
}

// nt is a multiple of K, so a thread's slots are equally spaced.
template <int K, bool CORR = true>
__device__ __forceinline__ void commit_tile(float2 *sx, float2 *sc, const TileRegs<K> &r, const Job &j, int M) {
  const int tid = threadIdx.x, step = lds_slot<K>(blockDim.x);
  float2 *p = sx + lds_slot<K>(tid);
  p[0] = j.first && tid < M - 1 ? make_float2(0.f, 0.f) : r.win[0];
#pragma unroll
  for (int u = 1; u < K; ++u) p[u * step] = r.win[u];
  if (tid < M - 1) {
    p[K * step] = r.win[K];
    if (CORR && j.head) sc[tid] = r.cv;
  }
}

// The tile's main arithmetic (window in sx) for this thread's K outputs.
// BC: largest Horner length compiled (10 or 16; fewer unrolled paths keep
// the register budget of the common configurations small).  MASKED: tiles
// may carry branch sets that are not prefixes (bit-mask control tokens).
template <int MT, int K, int BC, bool MASKED>
__device__ __forceinline__ void tile_compute(const float2 *sx, cfloat2p ht, const Job &j, int M, float (&ar)[K],
                                             float (&ai)[K]) {
  const int q0 = threadIdx.x * K;
#pragma unroll
  for (int k = 0; k < K; ++k) ar[k] = ai[k] = 0.f;
  if (q0 >= j.nout) return;
  switch (j.B) {
#define DF_CASE(n) \
  case n:                                                  \
    if constexpr (n <= BC) horner_taps<MT, K, n, MASKED>(ht, j.set, sx, q0, M, ar, ai); \
    break;
    DF_CASE(1) DF_CASE(2) DF_CASE(3) DF_CASE(4) DF_CASE(5) DF_CASE(6) DF_CASE(7) DF_CASE(8)
    DF_CASE(9) DF_CASE(10) DF_CASE(11) DF_CASE(12) DF_CASE(13) DF_CASE(14) DF_CASE(15) DF_CASE(16)
#undef DF_CASE
    default: break;
  }
}

// Where pair k of lane's outputs lies in a wavefront's part of the store
// buffer, in bytes: the pairs of the lanes whose outputs start on the same
// banks are exchanged against each other.
template <int K>
__device__ __forceinline__ uint32_t store_slot(uint32_t lane, int k) {
  constexpr uint32_t P = K / 2;
  return (lane * P + (lane / (16 / P)) % P) * 16 ^ (uint32_t)k * 16;
}

// Store this thread's outputs; in a firing's first tile, outputs q < M-1
// first add their head correction (staged in sc).
// A wavefront whose 64 K outputs are all there and start on 16 bytes passes
// them through its part of `so` (LDS, K * threads samples; null: not given), so
// that every store instruction writes one run of 1 KiB; stored from where they
// are formed, 16 bytes of each 8 K bytes at a time, they take the L2 K / 2
// requests for each run of 8 K bytes.  2^24 samples, 10 branches: 4 taps 73 and 65 us, 8 taps
// 78 and 72, 16 taps 109 and 108 (VALU-bound; the pass with push and pop 168
// and 161; 32 firings of 65536 with 10 taps 27.2 and 26.0).
template <int K>
__device__ __forceinline__ void tile_store(float4 *so, const float2 *sc, const Job &j, int M, float (&ar)[K],
                                           float (&ai)[K]) {
  const int q0 = threadIdx.x * K;
  if (q0 >= j.nout) return;
  if (j.head && q0 < M - 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int q = q0 + k;
      if (q < M - 1 && q < j.nout) {
        ar[k] += sc[q].x;
        ai[k] += sc[q].y;
      }
    }
  }
  int64_t slot;
  if (!ring_run(j.yb, j.y_mask, j.nout, &slot)) {
    char *p = (char *)(j.y + slot);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (so && (w + 1) * 64 * K <= j.nout && ((uintptr_t)p & 15) == 0) {   // uniform
      char *b = (char *)so + w * 512 * K, *q = p + (uint32_t)w * (512u * K);
      uint32_t l = threadIdx.x & 63;
      asm volatile("" : "+v"(l));                        // the offsets are formed here, not held across the tile
#pragma unroll
      for (int k = 0; k < K / 2; ++k)
        *(float4 *)(b + store_slot<K>(l, k)) = make_float4(ar[2 * k], ai[2 * k], ar[2 * k + 1], ai[2 * k + 1]);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // read by other lanes of the wavefront
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // pair 64 c + l is pair l % (K/2) of lane (64 c + l) / (K/2)
      const uint32_t from = store_slot<K>(l / (K / 2), l % (K / 2));
#pragma unroll
      for (int c = 0; c < K / 2; ++c)
        *(float4 *)(q + 16u * l + 1024u * c) = *(const float4 *)(b + from + 1024 * c);
      return;
    }
    const uint32_t off = (uint32_t)q0 * 8u;              // a multiple of 32
    if (q0 + K <= j.nout) {
      if (((uintptr_t)p & 15) == 0) {                    // uniform: pairs of outputs in 16-byte stores
#pragma unroll
        for (int k = 0; k < K; k += 2)
          *(float4 *)(p + off + 8 * k) = make_float4(ar[k], ai[k], ar[k + 1], ai[k + 1]);
      } else {
#pragma unroll
        for (int k = 0; k < K; ++k) *(float2 *)(p + off + 8 * k) = make_float2(ar[k], ai[k]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (q0 + k < j.nout) *(float2 *)(p + off + 8 * k) = make_float2(ar[k], ai[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (q0 + k < j.nout) j.y[(slot + q0 + k) & j.y_mask] = make_float2(ar[k], ai[k]);
  }
}

// Word w of a lane-distributed descriptor (lane w holds word w).
__device__ __forceinline__ uint32_t dword_at(uint32_t dv, int w) {
  return (uint32_t)__builtin_amdgcn_readlane((int)dv, w);
}
__device__ __forceinline__ uint64_t qword_at(uint32_t dv, int w) {
  return (uint64_t)dword_at(dv, w) | ((uint64_t)dword_at(dv, w + 1) << 32);
}

// A workgroup's tiles: blockIdx.x, + gridDim.x, ... < n_items.  Tiles come
// grouped by Horner length, longest first, so a compute unit whose workgroups
// all walk forwards is bound by arithmetic first and by memory last.  Every
// second workgroup of a compute unit (workgroups 256 apart share one of the
// 256 units) walks its own tiles backwards, so that long and short ones
// overlap all the time; which tiles a workgroup has does not change.
struct Walk {
  int64_t item, step, left;
  __device__ __forceinline__ bool start(int64_t n_items) {
    const int64_t b = blockIdx.x, g = gridDim.x;
    if (b >= n_items) return false;
    left = (uint64_t)(n_items - b + g - 1) / (uint32_t)g;
    const bool back = (blockIdx.x >> 8) & 1;
    item = back ? b + (left - 1) * g : b;
    step = back ? -g : g;
    return true;
  }
};

// The whole pipelined loop over a workgroup's tiles.
// src.fetch(k) loads tile k's raw descriptor two tiles ahead; src.expand(raw,
// job) turns it into the uniform Job when the tile's loads are issued.  A
// source with kOwnHeads forms a first tile's head corrections itself
// (src.heads, the whole workgroup, into sc).
// MT: the compiled tap count, or 0 (any count, Mr).
template <int MT, int K, int BC, bool MASKED, class Src>
__device__ __forceinline__ void run_tiles(float2 *sx, float2 *sc, float4 *so, int64_t n_items, Src &src, int Mr) {
  constexpr bool CORR = !Src::kOwnHeads;
  const int M = MT ? MT : Mr;
  Walk w;
  if (!w.start(n_items)) return;                     // uniform
  Job cur, nxt;
  src.expand(src.fetch(w.item), cur);
  TileRegs<K> regs;
  load_tile<K, CORR>(regs, cur, M);
  if (w.left > 1) src.expand(src.fetch(w.item + w.step), nxt);
  for (;;) {
    commit_tile<K, CORR>(sx, sc, regs, cur, M);
    if constexpr (Src::kOwnHeads) {
      if (cur.head) src.heads(sc, cur, M);
    }
    __syncthreads();
    if (w.left > 1) load_tile<K, CORR>(regs, nxt, M);
    typename Src::Raw nn{};
    if (w.left > 2) nn = src.fetch(w.item + 2 * w.step);
    float ar[K], ai[K];
    tile_compute<MT, K, BC, MASKED>(sx, as_const(cur.h), cur, M, ar, ai);
    if (w.left > 1) settle<K, CORR>(regs);
    tile_store<K>(so, sc, cur, M, ar, ai);
    if (w.left == 1) break;
    __syncthreads();
    w.item += w.step;
    cur = nxt;
    if (w.left > 2) src.expand(nn, nxt);
    --w.left;
  }
}

// ------------------------------------------------------------------ matrix cores
// Matrix-core form of a tile for M = 16 taps.  The per-tap polynomial is a
// matrix product: for a block of 16 window samples s and a chunk of four
// branches, Q[m][s] = sum_b h_b[m] p_s^b is one v_mfma_f32_16x16x4_f32
// (rows: taps m, columns: samples s, inner index: branches b; one product
// for the real and one for the imaginary part of h), accumulated over the
// ceil(B/4) chunks.  The rest stays on the VALU: Z[m][s] = x_s Q[m][s]
// (complex), and y[q] = sum_m Z[m][q + 15 - m] (window sample i = q + 15 - m
// for output q), taken in two steps.  Lane (row rho, column j) holds Z for
// taps 4 rho + r (r = 0..3, the product's accumulator layout) of sample j;
// shifting register r by r lanes inside the 16-lane row (DPP) aligns every
// value on lane u = j + r, so a row sums to
//   R_rho[16k + u] = sum_r Z[4 rho + r][16k + u - r]   (block k),
// with positions u >= 16 carried to the next block's first lanes.  Each
// R_rho is written to LDS, and after a barrier
//   y[q] = R_0[q + 15] + R_1[q + 11] + R_2[q + 7] + R_3[q + 3].
// The products are exact float products with float accumulation (the
// power-basis sum, not Horner's rule), so this form rounds differently from
// the VALU form; when it is selected (DFHIP_BODY=mx), every kernel that runs
// M = 16 bodies uses it, so the batching paths stay bit-identical.  On
// MI355X it is the slower form: the complex products, row combination,
// powers and LDS staging it leaves on the VALU cost nearly as many VALU
// instructions as Horner's rule (SQ_INSTS_VALU per launch 60 M + 4 M
// matrix products against 66 M), and the matrix products add latency.

typedef float mx4 __attribute__((ext_vector_type(4)));

// Lane i of a 16-lane row receives lane i-S of the same row (0 below the
// row start): one DPP move.
template <int S>
__device__ __forceinline__ float row_shr(float v) {
  if constexpr (S == 0) {
    return v;
  } else {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x110 + S, 0xF, 0xF, true));
  }
}

// Window and row-sum buffer sizes of a matrix-core tile (float2 slots): the
// blocks read window samples up to index tile + 30, and one block ahead.
template <int K>
__host__ __device__ constexpr int mx_window(int tile) { return lds_window<K>(tile + 48); }
__host__ __device__ constexpr int mx_row(int tile) { return tile + 32; }
template <int K>
__host__ __device__ constexpr int mx_lds(int tile) { return lds_corr(16) + mx_window<K>(tile) + 4 * mx_row(tile) + 256; }

// Coefficient operand of the tile's firing: lane l holds h_b[m] for branch
// b = 4c + l/16, tap m = l%16 (zero for branches outside the set).
struct MxCoef {
  float hr[4], hi[4];
};

// The operand passes through LDS (256 float2, written by wavefront 0 at the
// tile's commit), so that the block loop waits on LDS reads only, never on
// the next tile's global loads in flight.
__device__ __forceinline__ void mx_commit_coef(float2 *sh, const MxCoef &c) {
  if (threadIdx.x < 64) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sh[64 * k + threadIdx.x] = make_float2(c.hr[k], c.hi[k]);
  }
}

__device__ __forceinline__ void mx_read_coef(const float2 *sh, MxCoef &c) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float2 v = sh[64 * k + lane];
    c.hr[k] = v.x;
    c.hi[k] = v.y;
  }
}

template <bool MASKED>
__device__ __forceinline__ void mx_load_coef(MxCoef &c, const Job &j) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int b = 4 * k + (lane >> 4);
    const bool on = b < j.B && (!MASKED || in_set(j.set, b));
    const float2 v = on ? j.h[(lane & 15) * kCoefRow + b] : make_float2(0.f, 0.f);
    c.hr[k] = v.x;
    c.hi[k] = v.y;
  }
}

// Row sums of window block k for this wavefront's lanes: main (lane u:
// position 16k + u) and the part past the block end (lanes 0..2: positions
// 16k + 16 + u, carried into the next block).
template <int NCH>
__device__ __forceinline__ void mx_block(const float2 xv, const MxCoef &c, float &mr, float &mi, float &nr, float &ni) {
  const int rho = (threadIdx.x & 63) >> 4;
  const float p = fmaf(xv.x, xv.x, xv.y * xv.y);
  const float p2 = p * p;
  // p^(4c + rho): p^rho selected without branches, times p^4 per chunk
  float bp = ((rho & 1) ? p : 1.f) * ((rho & 2) ? p2 : 1.f);
  const float p4 = p2 * p2;
  mx4 qr = {0.f, 0.f, 0.f, 0.f}, qi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    qr = __builtin_amdgcn_mfma_f32_16x16x4f32(c.hr[ch], bp, qr, 0, 0, 0);
    qi = __builtin_amdgcn_mfma_f32_16x16x4f32(c.hi[ch], bp, qi, 0, 0, 0);
    if (ch + 1 < NCH) bp *= p4;
  }
  float zr[4], zi[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    zr[r] = fmaf(xv.x, qr[r], -(xv.y * qi[r]));
    zi[r] = fmaf(xv.x, qi[r], xv.y * qr[r]);
  }
  mr = zr[0] + row_shr<1>(zr[1]);
  mi = zi[0] + row_shr<1>(zi[1]);
  mr = mr + row_shr<2>(zr[2]);
  mi = mi + row_shr<2>(zi[2]);
  mr = mr + row_shr<3>(zr[3]);
  mi = mi + row_shr<3>(zi[3]);
  nr = row_shl<15>(zr[1]) + row_shl<14>(zr[2]);
  ni = row_shl<15>(zi[1]) + row_shl<14>(zi[2]);
  nr = nr + row_shl<13>(zr[3]);
  ni = ni + row_shl<13>(zi[3]);
}

// Blocks [k0, k1) of the tile for this wavefront (block k0 - 1 first, for
// the part of its row sums that falls into block k0).
template <int K, int NCH>
__device__ __forceinline__ void mx_blocks(const float2 *sx, float2 *rb, int rs, const MxCoef &c, int k0, int k1) {
  const int lane = threadIdx.x & 63, j = lane & 15, rho = lane >> 4;
  float cr = 0.f, ci = 0.f;                          // carried into lanes 0..2 from the block before
  if (k0 > 0) {
    float mr, mi;
    mx_block<NCH>(sx[lds_slot<K>(16 * (k0 - 1) + j)], c, mr, mi, cr, ci);
  }
  float2 *dst = rb + rho * rs + j;
  float2 xv = sx[lds_slot<K>(16 * k0 + j)];             // the next block's sample is read one block ahead
  for (int k = k0; k < k1; ++k) {
    const float2 xn = sx[lds_slot<K>(16 * (k + 1) + j)];
    float mr, mi, nr, ni;
    mx_block<NCH>(xv, c, mr, mi, nr, ni);
    dst[16 * k] = make_float2(mr + cr, mi + ci);
    cr = nr;
    ci = ni;
    xv = xn;
  }
}

// The tile's outputs q = threadIdx.x + NT*kk from the row sums (and the
// head corrections of a firing's first M-1 outputs).
template <int K>
__device__ __forceinline__ void mx_store(const float2 *sc, const float2 *rb, int rs, const Job &j) {
  const int nt = blockDim.x;
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    const int q = threadIdx.x + nt * kk;
    if (q >= j.nout) break;
    const float2 a = rb[q + 15], b = rb[rs + q + 11], c = rb[2 * rs + q + 7], d = rb[3 * rs + q + 3];
    float vr = a.x + b.x, vi = a.y + b.y;
    vr = vr + c.x;
    vi = vi + c.y;
    vr = vr + d.x;
    vi = vi + d.y;
    if (j.head && q < 15) {
      vr = vr + sc[q].x;
      vi = vi + sc[q].y;
    }
    j.y[(j.yb + q) & j.y_mask] = make_float2(vr, vi);
  }
}

// One tile on the matrix cores: the wavefronts split the tile's blocks,
// then every thread stores its outputs.
template <int K, int BC>
__device__ __forceinline__ void mx_tile(const float2 *sx, const float2 *sc, float2 *rb, const MxCoef &c, const Job &j) {
  const int rs = mx_row(K * (int)blockDim.x);
  const int nblk = (j.nout + 14) / 16 + 1;
  const int nw = blockDim.x >> 6, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k0 = nblk * w / nw, k1 = nblk * (w + 1) / nw;
  const int nch = (j.B + 3) >> 2;
  if (j.B > 0) {
    switch (nch) {
      case 1: mx_blocks<K, 1>(sx, rb, rs, c, k0, k1); break;
      case 2: mx_blocks<K, 2>(sx, rb, rs, c, k0, k1); break;
      case 3: mx_blocks<K, 3>(sx, rb, rs, c, k0, k1); break;
      default: if constexpr (BC > 12) mx_blocks<K, 4>(sx, rb, rs, c, k0, k1); break;
    }
  }
  __syncthreads();
  if (j.B > 0) {
    mx_store<K>(sc, rb, rs, j);
  } else {                                           // no active branch: zeros
    for (int q = threadIdx.x; q < j.nout; q += blockDim.x) j.y[(j.yb + q) & j.y_mask] = make_float2(0.f, 0.f);
  }
}

// The pipelined tile loop (as run_tiles) with matrix-core tiles (M = 16).
// LDS: [15] head corrections, window (mx_window), 4 row-sum rows (mx_row),
// coefficient operand (256).
template <int K, int BC, bool MASKED, class Src>
__device__ __forceinline__ void run_tiles_mx(float2 *sx, float2 *sc, float2 *rb, float2 *sh, int64_t n_items,
                                             Src &src) {
  constexpr int M = 16;
  Walk w;
  if (!w.start(n_items)) return;                     // uniform
  Job cur, nxt;
  src.expand(src.fetch(w.item), cur);
  TileRegs<K> regs;
  MxCoef cl;                                         // coefficient loads of the tile to commit
  load_tile<K>(regs, cur, M);
  mx_load_coef<MASKED>(cl, cur);
  if (w.left > 1) src.expand(src.fetch(w.item + w.step), nxt);
  for (;;) {
    commit_tile<K>(sx, sc, regs, cur, M);
    mx_commit_coef(sh, cl);
    __syncthreads();
    if (w.left > 1) {
      load_tile<K>(regs, nxt, M);
      mx_load_coef<MASKED>(cl, nxt);
    }
    typename Src::Raw nn{};
    if (w.left > 2) nn = src.fetch(w.item + 2 * w.step);
    MxCoef c;
    mx_read_coef(sh, c);
    mx_tile<K, BC>(sx, sc, rb, c, cur);
    if (w.left == 1) break;
    __syncthreads();
    w.item += w.step;
    cur = nxt;
    if (w.left > 2) src.expand(nn, nxt);
    --w.left;
  }
}

}  // namespace dfh
