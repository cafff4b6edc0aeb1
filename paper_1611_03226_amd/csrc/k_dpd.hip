// Predistortion actor body and batch commit.
//
// Actor body (Sec. 4.2: a polynomial actor feeding parallel FIR filters
// whose active set a configuration actor selects, summed by an adder):
//   y[t] = sum_{b<B} sum_{m<M} h[b][m] * psi_b(s_b[t-m]),  psi_b(x) = |x|^(2b) x.
// Inside a firing every active branch reads the same samples, so the sum is
// evaluated per tap as a polynomial in p = |x|^2 (Horner over branches):
//   y[t] = sum_m x[t-m] * P_m(p[t-m]),   P_m(p) = sum_{b<B} h[b][m] p^b.
// Only the first M-1 outputs of a firing reach back into branch histories,
// which differ per branch (history source firing prev_b(g), or carried
// state); those terms are added by a per-branch correction.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "common.h"
#include "dpd_tile.h"
#include "host_logic.h"
#include "scan_dev.h"

namespace dfh {

__device__ __forceinline__ int64_t prev_of(const DpdArgs &a, int b, int64_t g) {
  if (a.prev) return a.prev[(int64_t)b * a.prev_stride + g];
  return (g % a.seg_firings) ? g - 1 : -1;
}

// Input sample at offset ii (< 0) before the start of firing g, as branch b
// sees it: tail of its history firing, carried state, or zero.
__device__ __forceinline__ float2 hist_sample(const DpdArgs &a, int64_t Rx, int b, int64_t g,
                                              int64_t pf, int64_t ii) {
  if (pf >= 0) return a.x[(Rx + pf * a.r + a.r + ii) & a.x_mask];
  if (a.hist) return a.hist[b * (a.M - 1) + (a.M - 1) + ii];
  return make_float2(0.f, 0.f);
}

// ------------------------------------------------------------------ coefficients
// Tap-major coefficients (see kCoefRow) from [B_max][M]: by one workgroup of
// a head pass, or a launch of their own.
__device__ __forceinline__ void coef_rows(const float2 *h, float2 *ht, int B_max, int M) {
  for (int t = threadIdx.x; t < M * kCoefRow; t += blockDim.x) {
    const int m = t / kCoefRow, b = t % kCoefRow;
    ht[t] = b < B_max ? h[b * M + m] : make_float2(0.f, 0.f);
  }
}

__global__ __launch_bounds__(512) void k_coef_rows(const float2 *h, float2 *ht, int B_max, int M) {
  coef_rows(h, ht, B_max, M);
}

size_t coef_rows_bytes(int M) { return sizeof(float2) * kCoefRow * (size_t)M; }

hipError_t launch_coef_rows(const float2 *h, float2 *ht, int B_max, int M, hipStream_t s) {
  hipLaunchKernelGGL(k_coef_rows, dim3(1), dim3(512), 0, s, h, ht, B_max, M);
  return hipGetLastError();
}

// ------------------------------------------------------------------ commit
// Advance the channel indices by the batch's token counts and carry each
// branch's history: the last M-1 input samples of its last feeding firing.
// One workgroup (the body's last).
// last_of(b): the last feeding firing of branch b, -1 for none.
template <class LastOf>
__device__ __forceinline__ void dpd_commit_block(const DpdCommitArgs &a, LastOf last_of) {
  const int64_t Rx = a.x_idx[0];
  __syncthreads();
  const int L = a.M - 1;
  for (int t = threadIdx.x; t < a.B_max * L; t += blockDim.x) {
    const int b = t / L, k = t - b * L;
    const int64_t lf = last_of(b);
    if (lf >= 0) a.hist[b * L + k] = a.x[(Rx + lf * a.r + a.r - L + k) & a.x_mask];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.x_idx[0] = Rx + a.n_firings * a.r;
    a.ctrl_idx[0] += a.n_firings;
    a.y_idx[1] += a.n_firings * a.r;
    check_chan(a.x_idx, a.err);
    check_chan(a.ctrl_idx, a.err);
    check_chan(a.y_idx, a.err);
  }
}

// ------------------------------------------------------------------ heads
// Head corrections of every firing with B > 0, a row of RL lanes per firing:
// 16 for M = 4, 8, 16; for any other tap count (MT = 0) the fewest of 4, 8, 16
// and 32 that hold the M - 1 outputs, so that short histories share a
// workgroup (30000 firings of 40 samples, with 32 lanes always and now: one
// tap 28 and 7 us, 12 taps 74 and 52).  corr[g][q], q < M-1, is read by the
// tiled body.  With a group
// table (one segment) the wavefront also derives the history sources of its
// firings and writes their prev/off table entries: its firings lie
// in one 64-firing group, so a ballot of the group's feed flags per branch
// plus the group's entry (count and last feeder before it) gives them;
// with order_out it also writes the firings' processing slots.
template <int MT, int RL, bool TABLES>
__global__ __launch_bounds__(256) void k_dpd_heads(DpdArgs a) {
  static_assert(MT == 0 || RL == 16, "head_correction's rows");
  constexpr int NR = 64 / RL;                         // firings of the workgroup
  const int M = MT ? MT : a.M;
  // The workgroup's four wavefronts share its firings; wavefront w takes
  // branches w, w+4, w+8, w+12 (more wavefronts in flight, a quarter of the
  // serial work each); each branch's sum goes to LDS and one wavefront adds
  // them in increasing branch order, as a single pass would.
  __shared__ float2 part[kMaxBranches][64];
  if constexpr (TABLES) {
    if ((int)blockIdx.x < a.ahead_blocks) {          // the next batch's scan (whole workgroups)
      scan_dev::scan_group(a.ahead, (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                           (a.ahead.seg_firings + 63) / 64);
      return;
    }
  }
  const int64_t hb = a.head_block0 + (int64_t)blockIdx.x - a.ahead_blocks;
  if (a.err_ahead && hb == 0 && threadIdx.x == 0) {
    const int32_t e = *a.err_ahead;
    if (e) {
      if (a.err) atomicOr(a.err, e);
      *a.err_ahead = 0;
    }
  }
  if (a.fill_ht && hb == 0) coef_rows(a.h, a.ht, a.B_max, M);
  const int64_t g0 = hb * NR;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t Rx = a.x_idx ? as_const(a.x_idx)[0] : 0;
  const int lane = threadIdx.x & 63, row = lane / RL, i = lane % RL;
  const int64_t g = g0 + row;                         // this lane's firing
  int64_t pf[kMaxBranches / 4];                       // history sources of this wavefront's branches
  if constexpr (TABLES) {
    const int64_t G = g0 >> 6;
    const int64_t gl = G * 64 + lane;                 // lane's firing of the group
    const bool gin = gl < a.n_firings;
    const uint32_t Bl = gin ? (a.B ? (uint32_t)a.B[gl] : prefix_set(a.B_const)) : 0u;
    const uint64_t below_mask = (1ull << ((g0 & 63) + row)) - 1;
#pragma unroll
    for (int b = 0; b < kMaxBranches; ++b) {
      if ((b & 3) != w) continue;                     // uniform
      pf[b >> 2] = -1;
      if (b >= a.B_max) continue;
      const uint64_t bal = __ballot(gin && (a.hist_mode == 1 || in_set(Bl, b)));
      const int64_t gi = 2 * (G * a.B_max + b);
      const int64_t cnt0 = as_const(a.grp)[gi], last0 = as_const(a.grp)[gi + 1];
      const uint64_t below = bal & below_mask;
      pf[b >> 2] = below ? G * 64 + 63 - __clzll((long long)below) : last0;
      if (i == b % RL && g < a.n_firings) {
        const int64_t o = (int64_t)b * a.prev_stride + g;
        a.tab_prev[o] = pf[b >> 2];
        if (a.tab_off) a.tab_off[o] = a.r * (cnt0 + __popcll(below));
      }
    }
    if (a.order_out) {
      // processing slot of each of the firings: its length's first
      // slot in this group plus the firings of that length before it here
      const int NV = a.B_max + 1;
      const int Ll = gin ? set_len(Bl) : -1;
      for (int q = w; q < NR; q += 4) {
        const int lq = (int)(g0 & 63) + q;            // group lane of firing g0 + q
        if (g0 + q >= a.n_firings) break;             // uniform
        const uint32_t Sq = (uint32_t)__builtin_amdgcn_readlane((int)Bl, lq);
        const int Lq = set_len(Sq);
        const uint64_t bal = __ballot(Ll == Lq);
        if (lane == q) {
          const int64_t k = as_const(a.obase)[G * NV + Lq] + __popcll(bal & ((1ull << lq) - 1));
          a.order_out[2 * k] = (int32_t)(g0 + q);
          a.order_out[2 * k + 1] = (int32_t)Sq;
        }
      }
    }
  }
  if (M == 1) return;                                 // no history
  const auto B_of = [&](int r) {
    const int64_t gr = g0 + r;
    return gr < a.n_firings ? (a.B ? (uint32_t)a.B[gr] : prefix_set(a.B_const)) : 0u;
  };
  // branch b of this wavefront (its at-th) in the lane's row
  const auto src_of = [&](int r, int b, int at) {
    if constexpr (TABLES) return pf[at];
    else return prev_of(a, b, g0 + r);
  };
  const auto sample = [&](int r, int b, int64_t p, int q) {
    return hist_sample(a, Rx, b, g0 + r, p, (int64_t)q - (M - 1));
  };
  const auto emit = [&](int b, bool, float sr, float si) { part[b][lane] = make_float2(sr, si); };
  if constexpr (MT != 0)
    head_correction<MT, NR>(as_const(a.h), B_of, [&](int r, int b) { return src_of(r, b, b >> 2); }, sample, w, 4, emit);
  else
    head_correction_any<RL>(as_const(a.h), M, B_of, src_of, sample, w, emit);
  __syncthreads();
  const uint32_t set = B_of(row);
  if (w == 0 && i < M - 1 && set != 0u) {
    float cr = 0.f, ci = 0.f;
    for (int b = 0; b < kMaxBranches; ++b)
      if (in_set(set, b)) {
        cr += part[b][lane].x;
        ci += part[b][lane].y;
      }
    a.corr[g * (M - 1) + i] = make_float2(cr, ci);
  }
}

// Whether this workgroup is the launch's last to come here.  Every other
// workgroup has read the channel indices by then (it read them before), and
// the commit reads nothing another workgroup wrote, so relaxed counters
// suffice (a device-scope fence here would write back the L2).
// Increments of one word by the whole chip take about 13 ns each, one after
// the other: more than the work of short firings (4096 of 64 samples: body 53
// us, now 8; 30000 of 40, 16 taps: 105 and 53).  So a larger grid counts on kTicketGroups words first, each
// on a cache line of its own and fed by workgroups of one XCD, and the last of
// a group on the first word.  All words are left at zero for the next batch.
__device__ __forceinline__ bool last_workgroup(int32_t *ticket) {
  __shared__ int last;
  __syncthreads();
  if (threadIdx.x == 0) {
    const auto count = [](int32_t *p, int n) {
      if (__hip_atomic_fetch_add(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != n - 1) return false;
      __hip_atomic_store(p, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return true;
    };
    const int grid = (int)gridDim.x, of = (int)blockIdx.x % kTicketGroups;
    if (grid <= 4 * kTicketGroups) {
      last = count(ticket, grid);
    } else {
      last = count(ticket + (1 + of) * kTicketStride, (grid - of + kTicketGroups - 1) / kTicketGroups) &&
             count(ticket, kTicketGroups);
    }
  }
  __syncthreads();
  return last;
}

// ------------------------------------------------------------------ tiled
// Tile descriptors of a single actor's batch: tile k is tile k % tpf of the
// (k / tpf)-th firing in processing order (pairs (firing, branch set) from
// the scan, or firing order).
struct SingleSrc {
  static constexpr bool kOwnHeads = false;
  const DpdArgs &a;
  int64_t Rx, Wy;
  __device__ SingleSrc(const DpdArgs &a_)
      : a(a_), Rx(a_.x_idx ? as_const(a_.x_idx)[0] : 0), Wy(a_.y_idx ? as_const(a_.y_idx)[1] : 0) {}
  struct Raw {
    uint32_t g, set, tile;                           // firing, branch set, tile of the firing
  };
  // scalar loads: a vector load here would share the window loads' counter
  __device__ Raw fetch(int64_t it) const {
    const uint32_t k = (uint32_t)it / (uint32_t)a.tiles_per_firing;
    const uint32_t tile = (uint32_t)it - k * (uint32_t)a.tiles_per_firing;
    if (a.order) return {(uint32_t)as_const(a.order)[2 * (int64_t)k], (uint32_t)as_const(a.order)[2 * (int64_t)k + 1], tile};
    return {k, a.B ? (uint32_t)as_const(a.B)[k] : prefix_set(a.B_const), tile};
  }
  __device__ void expand(const Raw &q, Job &j) const {
    const int64_t g = q.g;
    const uint32_t set = q.set;
    const int64_t t0 = (int64_t)q.tile * a.tile;
    j.x = a.x;
    j.y = a.y;
    j.h = a.ht;
    j.corr = a.corr + g * (a.M - 1);
    j.x_mask = a.x_mask;
    j.y_mask = a.y_mask;
    j.xb = Rx + g * a.r + t0;
    j.yb = Wy + g * a.r + t0;
    j.nout = (int)min((int64_t)a.tile, a.r - t0);
    j.set = set;
    j.B = set_len(set);
    j.first = t0 == 0;
    j.head = (t0 == 0 && set != 0u && a.corr) ? 1 : 0;
  }
};

// Grid-stride loop over the batch's tiles in the length-grouped firing order,
// pipelined as run_tiles describes.  MT: the compiled tap count (4, 8, 16),
// or 0: any count, the taps a loop.
template <int MT, int K, int BC, bool MASKED>
__global__ __launch_bounds__(256, MT == 0 && BC == 10 ? 4 : 1) void k_dpd_tiled(DpdArgs a) {
  extern __shared__ float4 lds4[];  // outputs on their way to memory, [M-1] head corrections, window
  float2 *sc = (float2 *)lds4 + a.tile, *sx = sc + lds_corr(MT ? MT : a.M);
  SingleSrc src(a);
  run_tiles<MT, K, BC, MASKED>(sx, sc, lds4, a.n_firings * a.tiles_per_firing, src, a.M);
  if (a.ticket && last_workgroup(a.ticket))
    dpd_commit_block(a.commit, [&](int b) { return a.commit.last[b]; });
}

// ------------------------------------------------------------------ small batches
//
// A batch of at most 64 firings in one launch: every wavefront reads the
// batch's control tokens (lane = firing), so a ballot per branch gives every
// history source, table entry and last feeder; the workgroup of a firing's
// first tile forms its head corrections, the last workgroup commits.  A small
// batch is bound by launches and latency: 64 firings of 256 samples took scan,
// head pass and body 5 + 6 + 7 us and two kernel boundaries, here 10 us (a
// pass with push and pop 27 and 20.5 us).
struct SmallSrc {
  static constexpr bool kOwnHeads = true;
  const DpdArgs &a;
  int64_t Rx, Wy;
  uint32_t sets;          // lane g: branch set of firing g
  bool shared_hist;
  float2 *part;           // LDS [16][32]: a branch's part of each correction
  const float2 *hs;       // LDS [B_max][M] coefficients
  struct Raw {
    uint32_t g, tile;
  };
  __device__ Raw fetch(int64_t it) const {
    const uint32_t k = (uint32_t)it / (uint32_t)a.tiles_per_firing;
    return {k, (uint32_t)it - k * (uint32_t)a.tiles_per_firing};
  }
  __device__ void expand(const Raw &q, Job &j) const {
    const uint32_t set = (uint32_t)__builtin_amdgcn_readlane((int)sets, (int)q.g);
    const int64_t t0 = (int64_t)q.tile * a.tile;
    j.x = a.x;
    j.y = a.y;
    j.h = a.ht;
    j.corr = nullptr;
    j.x_mask = a.x_mask;
    j.y_mask = a.y_mask;
    j.xb = Rx + (int64_t)q.g * a.r + t0;
    j.yb = Wy + (int64_t)q.g * a.r + t0;
    j.nout = (int)min((int64_t)a.tile, a.r - t0);
    j.set = set;
    j.B = set_len(set);
    j.first = t0 == 0;
    j.head = t0 == 0 && set != 0u;
    j.g = (int)q.g;
  }
  // Firings (bits) that feed branch b.
  __device__ uint64_t fed(int b) const {
    const int lane = threadIdx.x & 63;
    return __ballot(lane < (int)a.n_firings && (shared_hist || in_set(sets, b)));
  }
  // Head corrections of firing j.g, as the head pass forms them (the same
  // sums in the same order): branch b by a row of lanes (16, or 32 for tap
  // counts that are not compiled in), lane i its history sample and output.
  template <int MT>
  __device__ void form(float2 *sc, const Job &j, int Mr) const {
    constexpr int RL = MT ? 16 : 32, ROWS = 64 / RL;
    const int M = MT ? MT : Mr, L = M - 1;
    const int lane = threadIdx.x & 63, row = lane / RL, i = lane % RL;
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t before = (1ull << j.g) - 1;
    for (int b0 = 0; b0 < j.B; b0 += nw * ROWS) {        // uniform
      const int b = b0 + w * ROWS + row;
      int pf = -1;
      for (int c = 0; c < j.B; ++c) {
        const uint64_t below = fed(c) & before;
        if (c == b) pf = below ? 63 - __clzll((long long)below) : -1;
      }
      float2 xv = make_float2(0.f, 0.f);
      if (b < j.B && in_set(j.set, b) && i < L)
        xv = pf >= 0 ? a.x[(Rx + (int64_t)pf * a.r + a.r - L + i) & a.x_mask] : a.hist[b * L + i];
      const float pp = fmaf(xv.x, xv.x, xv.y * xv.y);
      float pb = 1.f;
      for (int e = 0; e < j.B; ++e) pb = e < b ? pb * pp : pb;
      const float pr = pb * xv.x, pi = pb * xv.y;
      const float2 *hb = hs + (b < j.B ? b : 0) * M;
      float sr = 0.f, si = 0.f;
      if constexpr (MT != 0) {
        row_taps<MT, 1>(hb, pr, pi, sr, si);
      } else {
        for (int m = 1; m < M; ++m) {
          const int from = RL * row + ((L + i - m) & (RL - 1));
          const float vr = __shfl(pr, from), vi = __shfl(pi, from);
          if (m > i) {
            const float2 c = hb[m];
            sr = fmaf(c.x, vr, sr);
            sr = fmaf(-c.y, vi, sr);
            si = fmaf(c.x, vi, si);
            si = fmaf(c.y, vr, si);
          }
        }
      }
      if (b < j.B) part[b * 32 + i] = make_float2(sr, si);
    }
    __syncthreads();
    if ((int)threadIdx.x < L) {
      float cr = 0.f, ci = 0.f;
      for (int b = 0; b < j.B; ++b)
        if (in_set(j.set, b)) {
          cr += part[b * 32 + threadIdx.x].x;
          ci += part[b * 32 + threadIdx.x].y;
        }
      sc[threadIdx.x] = make_float2(cr, ci);
    }
  }
};

template <int MT>
struct SmallTiles : SmallSrc {
  __device__ void heads(float2 *sc, const Job &j, int M) const { form<MT>(sc, j, M); }
};

template <int MT, int K, int BC, bool MASKED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_dpd_small(DpdArgs a, ScanArgs c) {
  extern __shared__ float4 lds4[];  // outputs on their way to memory, [M-1] head corrections, window, [16][32] parts,
                                    // [B_max][M] coefficients
  const int M = MT ? MT : a.M;
  float2 *sc = (float2 *)lds4 + a.tile, *sx = sc + lds_corr(M), *part = sx + lds_window<K>(a.tile + M - 1), *hs = part + 16 * 32;
  const int lane = threadIdx.x & 63, n = (int)a.n_firings;
  bool bad = false;
  uint32_t set = 0u;
  if (lane < n) set = token_set(c.ctrl[(c.ctrl_pos + lane) & c.ctrl_mask], c.ctrl_mode, a.B_max, &bad);
  SmallTiles<MT> src{{a, as_const(a.x_idx)[0], as_const(a.y_idx)[1], set, c.hist_mode == 1, part, hs}};
  for (int t = threadIdx.x; t < a.B_max * M; t += blockDim.x) hs[t] = a.h[t];
  if (threadIdx.x < 64) {
    if (blockIdx.x == 0 && __ballot(bad) && lane == 0) atomicOr(c.err, (int32_t)kErrControl);
    for (int g = blockIdx.x; g < n; g += gridDim.x) {    // the tables of firing g (as the head pass writes them)
      const uint64_t before = (1ull << g) - 1;
      for (int b = 0; b < a.B_max; ++b) {
        const uint64_t below = src.fed(b) & before;
        if (lane == b) {
          c.prev_out[(int64_t)b * c.stride + g] = below ? 63 - __clzll((long long)below) : -1;
          c.off_out[(int64_t)b * c.stride + g] = a.r * __popcll(below);
        }
      }
      if (lane == g) c.B_out[g] = (int32_t)set;
    }
  }
  __syncthreads();
  run_tiles<MT, K, BC, MASKED>(sx, sc, lds4, a.n_firings * a.tiles_per_firing, src, a.M);
  if (!last_workgroup(a.ticket)) return;
  __shared__ int last[kMaxBranches];
  if (threadIdx.x < 64)
    for (int b = 0; b < a.B_max; ++b) {
      const uint64_t f = src.fed(b);
      if (lane == 0) last[b] = f ? 63 - __clzll((long long)f) : -1;
    }
  __syncthreads();
  dpd_commit_block(a.commit, [&](int b) { return (int64_t)last[b]; });
}

// The same loop with matrix-core tiles (M = 16).
template <int K, int BC, bool MASKED>
__global__ __launch_bounds__(256) void k_dpd_tiled_mx(DpdArgs a) {
  extern __shared__ float2 lds[];   // [15] head corrections, window, 4 row-sum rows, coefficients
  float2 *sc = lds, *sx = sc + lds_corr(16), *rb = sx + mx_window<K>(a.tile), *sh = rb + 4 * mx_row(a.tile);
  SingleSrc src(a);
  run_tiles_mx<K, BC, MASKED>(sx, sc, rb, sh, a.n_firings * a.tiles_per_firing, src);
  if (a.ticket && last_workgroup(a.ticket))
    dpd_commit_block(a.commit, [&](int b) { return a.commit.last[b]; });
}

template <int K, int BC, bool MASKED>
static hipError_t launch_tiled_mx(const DpdArgs &a0, hipStream_t s, int tile, const KTiming *t) {
  DpdArgs a = a0;
  a.tile = tile;
  a.tiles_per_firing = (int32_t)((a.r + tile - 1) / tile);
  const int threads = tile / K;
  const size_t lds = (size_t)mx_lds<K>(tile) * sizeof(float2);
  const int64_t items = a.n_firings * a.tiles_per_firing;
  if (items <= 0) return hipSuccess;
  const int64_t resident = resident_blocks((const void *)k_dpd_tiled_mx<K, BC, MASKED>, threads, lds);
  const int64_t blocks = items < resident ? items : resident;
  if (t)
    hipExtLaunchKernelGGL((k_dpd_tiled_mx<K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, t->start,
                          t->stop, 0, a);
  else
    hipLaunchKernelGGL((k_dpd_tiled_mx<K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <int MT, int K, int BC, bool MASKED>
static hipError_t launch_tiled(const DpdArgs &a0, hipStream_t s, int tile, const KTiming *t) {
  DpdArgs a = a0;
  a.tile = tile;
  a.tiles_per_firing = (int32_t)((a.r + tile - 1) / tile);
  const int threads = tile / K;
  const size_t lds = (size_t)(tile + lds_window<K>(tile + a.M - 1) + lds_corr(a.M)) * sizeof(float2);
  const int64_t items = a.n_firings * a.tiles_per_firing;
  if (items <= 0) return hipSuccess;
  const int64_t resident = resident_blocks((const void *)k_dpd_tiled<MT, K, BC, MASKED>, threads, lds);
  const int64_t blocks = items < resident ? items : resident;
  if (t)
    hipExtLaunchKernelGGL((k_dpd_tiled<MT, K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, t->start, t->stop,
                          0, a);
  else
    hipLaunchKernelGGL((k_dpd_tiled<MT, K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ samples
//
// One thread per output sample, for batches of firings (or rows) so short that
// a tile would leave most of its lanes idle, or so few that a launch counts
// (host::sample_wise has the figures).  Bound by VALU issue, and
// where firings are short by the corrections, which few lanes of a wavefront
// form.  No head pass: a sample that reaches before
// its firing forms its own correction.  Every sum is the tiled body's, in its
// order (zeros before the firing's start included), so the batches that take
// this kernel give the bits of those that do not.
// ROWS: every firing has all B_const branches and none before it.
template <bool ROWS>
__device__ __forceinline__ float2 sample_output(const DpdArgs &a, int64_t Rx, int64_t g, int64_t i) {
  const int M = a.M;
  const uint32_t set = ROWS ? prefix_set(a.B_const) : (uint32_t)a.B[g];
  const int B = ROWS ? a.B_const : set_len(set);
  int Bw = B;                                            // largest Horner length of the wavefront
  if constexpr (!ROWS) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) Bw = max(Bw, __shfl_xor(Bw, o));
    Bw = __builtin_amdgcn_readfirstlane(Bw);
  }
  const cfloat2p h = as_const(a.h);
  const int64_t at = Rx + g * a.r + i;
  float ar = 0.f, ai = 0.f;
  for (int m = 0; m < M; ++m) {
    const float2 xv = i >= m ? a.x[(at - m) & a.x_mask] : make_float2(0.f, 0.f);
    const float p = fmaf(xv.x, xv.x, xv.y * xv.y);
    float Pr = 0.f, Pi = 0.f;
    for (int b = Bw - 1; b >= 0; --b) {
      const float2 c = ldc(h, b * M + m);
      if constexpr (ROWS) {
        Pr = b == B - 1 ? c.x : fmaf(Pr, p, c.x);
        Pi = b == B - 1 ? c.y : fmaf(Pi, p, c.y);
      } else {                                           // branches outside the set: zeros
        const bool on = in_set(set, b);
        const float cx = on ? c.x : 0.f, cy = on ? c.y : 0.f;
        Pr = b >= B - 1 ? cx : fmaf(Pr, p, cx);
        Pi = b >= B - 1 ? cy : fmaf(Pi, p, cy);
      }
    }
    ar = fmaf(xv.x, Pr, ar);
    ar = fmaf(-xv.y, Pi, ar);
    ai = fmaf(xv.x, Pi, ai);
    ai = fmaf(xv.y, Pr, ai);
  }
  if constexpr (!ROWS) {
    if (i < M - 1 && set != 0u) {                        // the head correction, as the head pass forms it
      float cr = 0.f, ci = 0.f;
      for (int b = 0; b < B; ++b) {
        if (!in_set(set, b)) continue;
        const int64_t pf = prev_of(a, b, g);
        float sr = 0.f, si = 0.f;
        for (int m0 = 1; m0 < M; m0 += 4) {              // four terms' loads and powers at once
          float2 xv[4];
          float pp[4], pb[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            xv[j] = make_float2(0.f, 0.f);
            if (m0 + j > i && m0 + j < M) xv[j] = hist_sample(a, Rx, b, g, pf, i - (m0 + j));
            pp[j] = fmaf(xv[j].x, xv[j].x, xv[j].y * xv[j].y);
            pb[j] = 1.f;
          }
          for (int e = 0; e < b; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) pb[j] *= pp[j];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (m0 + j > i && m0 + j < M) {
              const float vr = pb[j] * xv[j].x, vi = pb[j] * xv[j].y;
              const float2 c = ldc(h, b * M + m0 + j);
              sr = fmaf(c.x, vr, sr);
              sr = fmaf(-c.y, vi, sr);
              si = fmaf(c.x, vi, si);
              si = fmaf(c.y, vr, si);
            }
        }
        cr += sr;
        ci += si;
      }
      ar += cr;
      ai += ci;
    }
  }
  return set ? make_float2(ar, ai) : make_float2(0.f, 0.f);   // (no branch: not 0 x infinity)
}

template <bool ROWS>
__global__ __launch_bounds__(256) void k_dpd_samples(DpdArgs a) {
  const int64_t Rx = a.x_idx ? as_const(a.x_idx)[0] : 0, Wy = a.y_idx ? as_const(a.y_idx)[1] : 0;
  const int64_t total = a.n_firings * a.r, all = (total + 255) / 256 * 256;   // whole wavefronts
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < all; t += (int64_t)gridDim.x * 256) {
    const int64_t tc = t < total ? t : total - 1;
    const int64_t g = total >> 32 ? tc / a.r : (int64_t)((uint32_t)tc / (uint32_t)a.r);
    const float2 v = sample_output<ROWS>(a, Rx, g, tc - g * a.r);
    if (t < total) a.y[(Wy + t) & a.y_mask] = v;
  }
  if (a.ticket && last_workgroup(a.ticket))
    dpd_commit_block(a.commit, [&](int b) { return a.commit.last[b]; });
}

hipError_t launch_dpd_samples(const DpdArgs &a, hipStream_t s, const KTiming *t) {
  if (a.n_firings <= 0) return hipSuccess;
  if (a.M < 1 || a.M > kMaxTaps || a.order || (a.B && !a.prev)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)std::min<int64_t>((a.n_firings * a.r + 255) / 256, host::kMaxThreads / 256));
#define DF_SAMPLES(rows)                                                                              \
  if (t)                                                                                              \
    hipExtLaunchKernelGGL(k_dpd_samples<rows>, grid, dim3(256), 0, s, t->start, t->stop, 0, a);       \
  else                                                                                                \
    hipLaunchKernelGGL(k_dpd_samples<rows>, grid, dim3(256), 0, s, a);
  if (a.B) {
    DF_SAMPLES(false)
  } else {
    DF_SAMPLES(true)
  }
#undef DF_SAMPLES
  return hipGetLastError();
}

template <int MT, int K, int BC, bool MASKED>
static hipError_t launch_small(const DpdArgs &a0, const ScanArgs &c, hipStream_t s, int tile, const KTiming *t) {
  DpdArgs a = a0;
  a.tile = tile;
  a.tiles_per_firing = (int32_t)((a.r + tile - 1) / tile);
  const int threads = tile / K;
  const size_t lds = (size_t)(tile + lds_window<K>(tile + a.M - 1) + lds_corr(a.M) + 16 * 32 + a.B_max * a.M) * sizeof(float2);
  const int64_t items = a.n_firings * a.tiles_per_firing;
  const int64_t resident = resident_blocks((const void *)k_dpd_small<MT, K, BC, MASKED>, threads, lds);
  const int64_t blocks = items < resident ? items : resident;
  if (t)
    hipExtLaunchKernelGGL((k_dpd_small<MT, K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, t->start,
                          t->stop, 0, a, c);
  else
    hipLaunchKernelGGL((k_dpd_small<MT, K, BC, MASKED>), dim3((unsigned)blocks), dim3(threads), lds, s, a, c);
  return hipGetLastError();
}

bool dpd_body_mx_env() {
  const char *v = getenv("DFHIP_BODY");
  return v && strcmp(v, "mx") == 0;
}

hipError_t launch_dpd_heads(const DpdArgs &a, hipStream_t s) {
  if (a.n_firings <= 0) return hipSuccess;
  if (!a.corr || a.M < 1 || a.M > kMaxTaps || (a.fill_ht && !a.ht)) return hipErrorInvalidValue;
  if (a.grp && (a.seg_firings != a.n_firings || !a.tab_prev)) return hipErrorInvalidValue;
  if (a.ahead_blocks < 0 || (a.ahead_blocks && (!a.grp || a.ahead.n_segs != 1 || !a.ahead.grp || !a.ahead.ticket ||
                                               a.ahead_blocks != (scan_groups(1, a.ahead.seg_firings) + 3) / 4)))
    return hipErrorInvalidValue;
  const int rl = host::head_lanes(a.M);
  const int nr = 64 / rl;                              // firings per workgroup
  // in pieces that a grid can hold beside the scan's workgroups
  const int64_t blocks = (a.n_firings + nr - 1) / nr, most = host::kMaxThreads / 512;
  for (DpdArgs p = a; p.head_block0 < blocks; p.head_block0 += most, p.ahead_blocks = 0) {
    const dim3 grid((unsigned)(std::min(blocks - p.head_block0, most) + p.ahead_blocks));
#define DF_HEADS(m, l)                                                                  \
  if ((m == 0 || a.M == m) && rl == l) {                                                \
    if (a.grp)                                                                          \
      hipLaunchKernelGGL((k_dpd_heads<m, l, true>), grid, dim3(256), 0, s, p);          \
    else                                                                                \
      hipLaunchKernelGGL((k_dpd_heads<m, l, false>), grid, dim3(256), 0, s, p);         \
  }
    DF_HEADS(16, 16) else DF_HEADS(8, 16) else DF_HEADS(4, 16)
    else DF_HEADS(0, 4) else DF_HEADS(0, 8) else DF_HEADS(0, 16) else DF_HEADS(0, 32)
#undef DF_HEADS
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

static host::TileShape tile_shape(const DpdArgs &a, int tile, int outputs_per_thread) {
  return host::tile_shape(a.n_firings, a.r, a.M == 16 && a.mx, tile, outputs_per_thread);
}

hipError_t launch_dpd_small(const DpdArgs &a, const ScanArgs &c, hipStream_t s, int tile, int outputs_per_thread,
                            const KTiming *t) {
  if (a.n_firings < 1 || a.n_firings > 64 || !a.ht || !a.h || !a.hist || !a.x_idx || !a.y_idx || !a.ticket || !c.ctrl ||
      !c.B_out || !c.prev_out || !c.off_out || !c.err || a.M < 1 || a.M > kMaxTaps)
    return hipErrorInvalidValue;
  const host::TileShape sh = tile_shape(a, tile, outputs_per_thread);
  const bool small = a.B_max <= 10;
#define DF_SMALL(m, k)                                                                       \
  if ((m == 0 || a.M == m) && sh.K == k)                                                     \
    return a.masked ? launch_small<m, k, 16, true>(a, c, s, sh.tile, t)                      \
                    : (small ? launch_small<m, k, 10, false>(a, c, s, sh.tile, t)            \
                             : launch_small<m, k, 16, false>(a, c, s, sh.tile, t));
  DF_SMALL(16, 4) DF_SMALL(16, 8) DF_SMALL(8, 4) DF_SMALL(8, 8) DF_SMALL(4, 4) DF_SMALL(4, 8)
  DF_SMALL(0, 4) DF_SMALL(0, 8)
#undef DF_SMALL
  return hipErrorInvalidValue;
}

hipError_t launch_dpd_body(const DpdArgs &a, hipStream_t s, int tile, int outputs_per_thread, const KTiming *t) {
  if (a.n_firings <= 0) return hipSuccess;
  if (!a.ht || a.M < 1 || a.M > kMaxTaps) return hipErrorInvalidValue;
  const host::TileShape sh = tile_shape(a, tile, outputs_per_thread);
  const int K = sh.K, tl = sh.tile;
  // compiled paths: Horner lengths up to 10 or up to 16; branch sets that are
  // not prefixes (bit-mask tokens) take the masked paths up to 16
  const bool small = a.B_max <= 10;
  if (a.M == 16 && a.mx) {
    if (K == 4)
      return a.masked ? launch_tiled_mx<4, 16, true>(a, s, tl, t)
                      : (small ? launch_tiled_mx<4, 10, false>(a, s, tl, t) : launch_tiled_mx<4, 16, false>(a, s, tl, t));
    return a.masked ? launch_tiled_mx<8, 16, true>(a, s, tl, t)
                    : (small ? launch_tiled_mx<8, 10, false>(a, s, tl, t) : launch_tiled_mx<8, 16, false>(a, s, tl, t));
  }
#define DF_TILED(m, k)                                                                      \
  if ((m == 0 || a.M == m) && K == k)                                                       \
    return a.masked ? launch_tiled<m, k, 16, true>(a, s, tl, t)                             \
                    : (small ? launch_tiled<m, k, 10, false>(a, s, tl, t) : launch_tiled<m, k, 16, false>(a, s, tl, t));
  DF_TILED(16, 4) DF_TILED(16, 8) DF_TILED(8, 4) DF_TILED(8, 8) DF_TILED(4, 4) DF_TILED(4, 8)
  DF_TILED(0, 4) DF_TILED(0, 8)
#undef DF_TILED
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ small helpers
__global__ void k_advance(int64_t *idx, int64_t delta, int32_t *err) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    idx[0] += delta;
    check_chan(chan_slot(idx), err);
  }
}

hipError_t launch_advance(int64_t *idx, int64_t delta, int32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, idx, delta, err);
  return hipGetLastError();
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

}  // namespace dfh
