// Adjoints for coefficient adaptation through a memory-polynomial PA.
//
// Gradients use the real-pair convention: for complex z, dL/dRe z + i dL/dIm z.
//
// Coefficient adjoint of the predistortion actor (y linear in h):
//   grad_h[b][m] = sum_n G[n] conj(psi_b(s_b[n-m])),  b < B of n's firing.
// Inside a firing the source sample is branch independent, so with
// z = G[n] conj(x[n-m]) and p = |x[n-m]|^2 each (n, m) pair feeds all
// branches through the running power z p^b.  Taps reaching before a firing
// start read branch b's own history and are added per branch.
// Reduction: fp32 partial sums per workgroup in a fixed order, then an fp64
// sum over workgroups in a fixed order (deterministic, no float atomics).
//
// Input adjoint of v[n] = sum_k sum_q a[k][q] phi_k(u[n-q]),
// phi_k(u) = |u|^(2k) u: with d phi/du = (k+1) p^k and
// d phi/du* = k p^(k-1) u^2 (p = |u|^2),
//   Gu[n] = sum_q g[n+q] conj(A_q) + conj(g[n+q]) Bw_q u^2,
//   A_q = sum_k a[k][q] (k+1) p^k,  Bw_q = sum_{k>=1} a[k][q] k p^(k-1).
#include <algorithm>

#include "common.h"
#include "dpd_tile.h"

namespace dfh {


__device__ __forceinline__ int64_t adj_prev(const AdjArgs &a, int b, int64_t g) {
  if (a.prev) return a.prev[(int64_t)b * a.prev_stride + g];
  return (g % a.seg_firings) ? g - 1 : -1;
}

// Lane reduce-scatter of N values per lane over the 64 lanes of a
// wavefront, in six steps; step k pairs each lane with a partner that
// differs in lane bit 32 >> k (and agrees in the bits split before): the
// lane with that bit set keeps the upper half of its values (padded to an
// even count with zeros), the other the lower half, each adding the
// partner's copy.  Steps 0 and 1 pair lanes 32 and 16 apart with the
// permlane swaps (a swap and an add per kept value); steps 2..5 use the
// DPP row mirror (lane 15 - l), half-row mirror (7 - l) and quad
// permutations (l ^ 2, l ^ 1) as partners (two selects and an add).  The
// partners' lane masks 32, 16, 15, 7, 2, 1 are independent, so after the
// six steps every kept value is summed over all 64 lanes exactly once, in
// a fixed order.
constexpr int rs_half(int n) { return (n + 1) / 2; }

template <int STEP, int N, int CAP>
__device__ __forceinline__ void rs_steps(float (&v)[CAP], int lane) {
  constexpr int H = rs_half(N);
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const float lo = v[i];
    const float hi = i + H < N ? v[i + H] : 0.f;
    if constexpr (STEP < 2) {
      const auto sw = STEP == 0 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false)
                                : __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
      v[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    } else {
      constexpr int ctrl = STEP == 2 ? 0x140 : STEP == 3 ? 0x141 : STEP == 4 ? 0x4E : 0xB1;
      const bool up = (lane & (32 >> STEP)) != 0;
      const float send = up ? lo : hi, keep = up ? hi : lo;
      v[i] = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), ctrl, 0xF, 0xF, false));
    }
  }
  if constexpr (STEP < 5) rs_steps<STEP + 1, H>(v, lane);
}

// Values a lane holds after the six steps, and the original index of its
// j-th one (-1 for padding).
template <int N>
struct RsPlan {
  static constexpr int n0 = N, n1 = rs_half(n0), n2 = rs_half(n1), n3 = rs_half(n2), n4 = rs_half(n3),
                       n5 = rs_half(n4), kept = rs_half(n5);
  __device__ static int index(int j, int lane) {
    const int cnt[6] = {n0, n1, n2, n3, n4, n5};
    int t = j;
    bool ok = true;
    for (int k = 5; k >= 0; --k) {
      if (lane & (32 >> k)) t += rs_half(cnt[k]);
      ok = ok && t < cnt[k];
    }
    return ok ? t : -1;
  }
};

// Taps per wavefront of the coefficient adjoint for BM branches (8 taps,
// with twice the accumulators and half the wavefronts per SIMD, measured
// slower at 10 branches).
constexpr int adj_tpw(int) { return 4; }

// One workgroup per (firing, span of input samples); one wavefront per
// group of TPW taps.  Every (sample, output) pair with the output in the
// firing is counted by the workgroup that owns the sample (pairs with a
// sample before the firing start are added at the end from the branch
// histories).  The span is processed in chunks of four samples per thread
// staged in LDS with the G values of the outputs they reach, and lane l of
// a wavefront takes samples l, l+64, ... of each chunk.  For its sample a
// lane forms p^b once and accumulates G[s+m] conj(x_s) p^b into TPW taps x
// BM branches of independent registers; after the span the wavefront
// reduces over lanes (fixed order).  The next chunk's loads are in flight
// (in registers) while the current one is processed; a chunk's G window
// starts with the last M+TPW-2 values of the previous one.
template <int BM, int TPW>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(BM <= 10 ? 4 : 1))) void k_adj_partial(
    AdjArgs a) {
  extern __shared__ float2 lds[];
  const int M = a.M;
  const int64_t g = blockIdx.x / a.blocks_per_firing;
  const int64_t c = blockIdx.x - g * a.blocks_per_firing;
  const int64_t s0 = c * a.span;
  const int64_t s1 = min(s0 + a.span, a.r);
  const uint32_t set = a.B ? (uint32_t)a.B[g] : prefix_set(BM);
  const int B = set_len(set);
  const int64_t xb = g * a.r;
  // chunk of C samples at n0: sx[i] = x[n0+i] (zero past the span), sg[o] =
  // G[n0+o] for o < C+K (zero past the firing); K = M+TPW-2 covers the taps
  // of the last wavefront's group past M, whose sums are dropped
  const int nt = blockDim.x, tid = threadIdx.x;
  const int C = a.chunk;                  // 4 * nt, a multiple of 64
  const int K = M + TPW - 2;
  float2 *sx = lds;
  float2 *sg = lds + C;
  float2 *red = sg + C + K;               // [BM][M] reduced sums
  const int lane = threadIdx.x & 63;
  const int m0 = (threadIdx.x >> 6) * TPW;  // first tap of this wavefront
  constexpr int NV = 2 * TPW * BM;        // TPW taps x BM branches x (re, im)
  float v[NV];                            // v[q*2BM + 2b + c]
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = 0.f;
  float2 carry = make_float2(0.f, 0.f);   // sg[tid] (tid < K) of the next chunk
  if (tid < K && s0 + tid < a.r) carry = a.G[xb + s0 + tid];
  float2 rx[4], rg[4];                    // the next chunk's x[n0 + j*nt + tid], G[n0 + K + j*nt + tid]
  const auto fetch = [&](int64_t n0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t n = n0 + j * nt + tid;
      rx[j] = n < s1 ? a.x[xb + n] : make_float2(0.f, 0.f);
      rg[j] = n + K < a.r ? a.G[xb + n + K] : make_float2(0.f, 0.f);
    }
  };
  fetch(s0);
  for (int64_t n0 = s0; n0 < s1; n0 += C) {
    if (tid < K) sg[tid] = carry;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sx[j * nt + tid] = rx[j];
      sg[K + j * nt + tid] = rg[j];
    }
    __syncthreads();
    if (n0 + C < s1) fetch(n0 + C);
    // sample n0 + i, output n0 + i + m
#pragma unroll 2
    for (int i = lane; i < C; i += 64) {
      const float2 xv = sx[i];
      const float p = fmaf(xv.x, xv.x, xv.y * xv.y);
      float pw[BM];
      pw[0] = 1.f;
#pragma unroll
      for (int b = 1; b < BM; ++b) pw[b] = pw[b - 1] * p;
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
        const float2 gv = sg[i + m0 + q];
        const float zr = fmaf(gv.x, xv.x, gv.y * xv.y);     // G conj(x)
        const float zi = fmaf(gv.y, xv.x, -(gv.x * xv.y));
#pragma unroll
        for (int b = 0; b < BM; ++b) {
          v[q * 2 * BM + 2 * b] = fmaf(zr, pw[b], v[q * 2 * BM + 2 * b]);
          v[q * 2 * BM + 2 * b + 1] = fmaf(zi, pw[b], v[q * 2 * BM + 2 * b + 1]);
        }
      }
    }
    if (tid < K) carry = sg[C + tid];    // read before anyone rewrites the window
    __syncthreads();
  }
  rs_steps<0, NV>(v, lane);
#pragma unroll
  for (int j = 0; j < RsPlan<NV>::kept; ++j) {
    const int idx = RsPlan<NV>::index(j, lane);
    if (idx < 0) continue;
    const int q = idx / (2 * BM), rem = idx - q * 2 * BM;
    if (m0 + q < M) reinterpret_cast<float *>(&red[(rem >> 1) * M + m0 + q])[rem & 1] = v[j];
  }
  // taps before the firing start read branch b's history source: the last
  // M-1 samples of its previous feeding firing (zeros if none), staged in
  // LDS by all threads at once
  float2 *hx = red + BM * M;              // [BM][M-1]
  if (s0 == 0) {
    for (int t = threadIdx.x; t < B * (M - 1); t += blockDim.x) {
      const int b = t / (M - 1), i = t - b * (M - 1);
      const int64_t pf = adj_prev(a, b, g);
      hx[t] = pf >= 0 ? a.x[pf * a.r + a.r - (M - 1) + i] : make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < BM * M; t += blockDim.x) {
    const int b = t / M, mm = t - b * M;
    float sr = 0.f, si = 0.f;
    if (in_set(set, b)) {
      sr = red[t].x;
      si = red[t].y;
      if (s0 == 0) {
        // output i, tap mm reads history sample i - mm (< 0)
        for (int i = 0; i < mm && i < a.r; ++i) {
          const float2 xv = hx[b * (M - 1) + (M - 1) + i - mm];
          const float pp = fmaf(xv.x, xv.x, xv.y * xv.y);
          float pb = 1.f;
          for (int e = 0; e < b; ++e) pb *= pp;
          const float2 gv = a.G[xb + i];
          const float xr = pb * xv.x, xi = pb * xv.y;
          sr += gv.x * xr + gv.y * xi;
          si += gv.y * xr - gv.x * xi;
        }
      }
    }
    a.partial[(int64_t)t * gridDim.x + blockIdx.x] = make_float2(sr, si);
  }
}

// grad_h[b][m] = fp64 sum of the workgroup partials (stored [b][m][block]),
// fixed order: one workgroup per (b, m); thread t sums blocks t, t+256, ...,
// then a butterfly over each wavefront's lanes and the four wavefronts in
// order.
__global__ __launch_bounds__(256) void k_adj_reduce(const float2 *partial, int64_t n_blocks, float2 *grad) {
  __shared__ double wr[4], wi[4];
  const int e = blockIdx.x;               // b * M + m
  const float2 *src = partial + (int64_t)e * n_blocks;
  double ar = 0.0, ai = 0.0;
  int64_t k = threadIdx.x;
  for (; k + 768 < n_blocks; k += 1024) {  // four loads in flight
    const float2 v0 = src[k], v1 = src[k + 256], v2 = src[k + 512], v3 = src[k + 768];
    ar += v0.x;
    ai += v0.y;
    ar += v1.x;
    ai += v1.y;
    ar += v2.x;
    ai += v2.y;
    ar += v3.x;
    ai += v3.y;
  }
  for (; k < n_blocks; k += 256) {
    const float2 v = src[k];
    ar += v.x;
    ai += v.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ar += __shfl_xor(ar, o);
    ai += __shfl_xor(ai, o);
  }
  if ((threadIdx.x & 63) == 0) wr[threadIdx.x >> 6] = ar, wi[threadIdx.x >> 6] = ai;
  __syncthreads();
  if (threadIdx.x == 0)
    grad[e] = make_float2((float)(((wr[0] + wr[1]) + wr[2]) + wr[3]), (float)(((wi[0] + wi[1]) + wi[2]) + wi[3]));
}

hipError_t launch_adj(const AdjArgs &a, hipStream_t s) {
  const int64_t blocks = a.n_firings * a.blocks_per_firing;
  if (blocks > 0) {
    // one wavefront per adj_tpw(B_max) taps; chunks of four samples per
    // thread; LDS: samples, G window, reduced sums, history samples
    AdjArgs b = a;
    const auto lds_of = [&](int threads, int tpw) {
      b.chunk = 4 * threads;
      return sizeof(float2) * ((size_t)2 * b.chunk + (a.M + tpw - 2) + (size_t)a.B_max * (2 * a.M - 1));
    };
    switch (a.B_max) {
#define DF_CASE(n)                                                                                  \
  case n: {                                                                                         \
    const int threads = 64 * ((a.M + adj_tpw(n) - 1) / adj_tpw(n));                                 \
    const size_t lds = lds_of(threads, adj_tpw(n));                                                 \
    hipLaunchKernelGGL((k_adj_partial<n, adj_tpw(n)>), dim3((unsigned)blocks), dim3(threads), lds, s, b); \
  } break;
      DF_CASE(1) DF_CASE(2) DF_CASE(3) DF_CASE(4) DF_CASE(5) DF_CASE(6) DF_CASE(7) DF_CASE(8)
      DF_CASE(9) DF_CASE(10) DF_CASE(11) DF_CASE(12) DF_CASE(13) DF_CASE(14) DF_CASE(15) DF_CASE(16)
#undef DF_CASE
      default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_adj_reduce, dim3(a.B_max * a.M), dim3(256), 0, s, a.partial, blocks, a.grad);
  return hipGetLastError();
}

// ------------------------------------------------------------------ amplifier model
//
// Forward with loss and input adjoint of the memory polynomial, in two forms.
// Runs: a workgroup takes a run of one row, a thread four consecutive samples
// of it: with four orders and four taps (the model in use) the thread's window
// sits in registers, the sixteen coefficients in scalar registers, and
// everything moves in 16-byte accesses; samples whose taps cross the row's end
// go sample by sample.  HBM-bound at 2^22 samples: the loss reads u and x and
// writes e (100 MB, 22 us), the adjoint reads u and g and writes Gu (100 MB, 20
// us, 32 us with a thread per sample that reloaded its coefficients and formed
// the powers per tap).
// Sample-wise, for any orders and taps and any rows: consecutive lanes take
// consecutive samples of the batch, so every access of a tap is one contiguous
// run, and a thread's U samples share the coefficients' scalar loads.  Bound by
// VALU and the scalar loads' latency, so U grows with the batch.  us of the
// adjoint with four consecutive samples a thread / a sample a thread / now, and
// of the loss with four consecutive / now: 5 orders, 4 taps, 2^22 samples 56 /
// 37 / 27, 61 / 31; 8 orders, 16 taps 160 / 151 / 98, 164 / 78; 20000 rows of
// 40 samples, 4 and 4 29 / 8.7 / 6.9, 53 / 11.
typedef float f4_any __attribute__((ext_vector_type(4), aligned(8)));

__device__ __forceinline__ void load4(const float2 *p, float2 (&v)[4]) {
  const f4_any a = *(const f4_any *)p, b = *(const f4_any *)(p + 2);
  v[0] = make_float2(a.x, a.y), v[1] = make_float2(a.z, a.w);
  v[2] = make_float2(b.x, b.y), v[3] = make_float2(b.z, b.w);
}

__device__ __forceinline__ void store4(float2 *p, const float2 (&v)[4]) {
  *(f4_any *)p = f4_any{v[0].x, v[0].y, v[1].x, v[1].y};
  *(f4_any *)(p + 2) = f4_any{v[2].x, v[2].y, v[3].x, v[3].y};
}

// Tap q's polynomial at p: P = sum_k a[k][q] p^k, and with DERIV its
// derivative D = sum_{k>=1} k a[k][q] p^(k-1) (Horner for both), for U values
// of p at once (the coefficients are the same).
template <bool DERIV, int U>
__device__ __forceinline__ void tap_polys(cfloat2p a, int K, int Q, int q, const float (&p)[U], float2 (&P)[U],
                                          float2 (&D)[U]) {
  const float2 top = ldc(a, (K - 1) * Q + q);
#pragma unroll
  for (int u = 0; u < U; ++u) P[u] = top, D[u] = make_float2(0.f, 0.f);
  for (int k = K - 2; k >= 0; --k) {
    const float2 c = ldc(a, k * Q + q);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (DERIV) D[u] = make_float2(fmaf(D[u].x, p[u], P[u].x), fmaf(D[u].y, p[u], P[u].y));
      P[u] = make_float2(fmaf(P[u].x, p[u], c.x), fmaf(P[u].y, p[u], c.y));
    }
  }
}

template <bool DERIV>
__device__ __forceinline__ void tap_poly(cfloat2p a, int K, int Q, int q, float p, float2 &P, float2 &D) {
  const float pp[1] = {p};
  float2 Pp[1], Dp[1];
  tap_polys<DERIV, 1>(a, K, Q, q, pp, Pp, Dp);
  P = Pp[0], D = Dp[0];
}

__device__ __forceinline__ float norm2(float2 v) { return fmaf(v.x, v.x, v.y * v.y); }

__device__ __forceinline__ void add_product(float2 &s, float2 x, float2 y) {   // s += x y
  s.x = fmaf(x.x, y.x, fmaf(-x.y, y.y, s.x));
  s.y = fmaf(x.x, y.y, fmaf(x.y, y.x, s.y));
}

// v[n] of a row.
__device__ __forceinline__ float2 mp_value(const float2 *u, cfloat2p a, int64_t n, int K, int Q) {
  float2 v = make_float2(0.f, 0.f), P, D;
  for (int q = 0; q < Q && q <= n; ++q) {
    const float2 w = u[n - q];
    tap_poly<false>(a, K, Q, q, norm2(w), P, D);
    add_product(v, w, P);
  }
  return v;
}

// One tap's part of Gu: g conj(A) + conj(g) D u^2 with A = P + p D.
__device__ __forceinline__ void add_adjoint(float2 &G, float2 g, float2 P, float2 D, float p, float2 u2) {
  const float2 A = make_float2(fmaf(p, D.x, P.x), fmaf(p, D.y, P.y));
  float2 w = make_float2(0.f, 0.f);
  add_product(w, D, u2);
  G.x = fmaf(g.x, A.x, fmaf(g.y, A.y, G.x));
  G.y = fmaf(g.y, A.x, fmaf(-g.x, A.y, G.y));
  G.x = fmaf(g.x, w.x, fmaf(g.y, w.y, G.x));
  G.y = fmaf(g.x, w.y, fmaf(-g.y, w.x, G.y));
}

__device__ __forceinline__ float2 square(float2 u) { return make_float2(u.x * u.x - u.y * u.y, 2.f * u.x * u.y); }

// Gu[n] of a row, without the scale of g.
__device__ __forceinline__ float2 mp_adjoint(float2 uv, const float2 *g, cfloat2p a, int64_t n, int64_t len, int K,
                                             int Q) {
  float2 G = make_float2(0.f, 0.f), P, D;
  const float p = norm2(uv);
  const float2 u2 = square(uv);
  for (int q = 0; q < Q && n + q < len; ++q) {
    tap_poly<true>(a, K, Q, q, p, P, D);
    add_adjoint(G, g[n + q], P, D, p, u2);
  }
  return G;
}

// The workgroup's sum of every thread's `sum`, in a fixed order.
__device__ __forceinline__ void block_sum(double sum, double (&ws)[4], double *out) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) sum += ws[w];
    out[blockIdx.x] = sum;
  }
}

// Runs of 1024 samples: run i is run i % runs_per_row of row
// i / runs_per_row; workgroups stride over them.
// k_mp_loss: e = v - x (stored when e is given) and per workgroup the sum of
// |e|^2 (each thread's in fp32 over its four samples, the rest in fp64).
__global__ __launch_bounds__(256) void k_mp_loss(MpArgs m, int64_t runs, int64_t runs_per_row) {
  __shared__ double ws[4];
  const cfloat2p a = as_const(m.a);
  double sum = 0.0;
  for (int64_t i = blockIdx.x; i < runs; i += gridDim.x) {
    const int64_t row = i / runs_per_row;
    const int64_t n0 = ((i - row * runs_per_row) * 256 + threadIdx.x) * 4;
    const float2 *u = m.u + row * m.len, *x = m.x + row * m.len;
    float2 *e = m.out ? m.out + row * m.len : nullptr;
    float part = 0.f;
    if (n0 >= 4 && n0 + 4 <= m.len) {
      float2 h[4], c[4], w[7], xv[4];
      load4(u + n0 - 4, h);
      load4(u + n0, c);
      load4(x + n0, xv);
#pragma unroll
      for (int j = 0; j < 7; ++j) w[j] = j < 3 ? h[j + 1] : c[j - 3];     // sample n0 - 3 + j
      float2 v[4], P, D;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = make_float2(-xv[k].x, -xv[k].y);
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        const float p = norm2(w[j]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = j - 3 + q;                                         // output n0 + k
          if (k < 0 || k > 3) continue;
          tap_poly<false>(a, 4, 4, q, p, P, D);
          add_product(v[k], w[j], P);
        }
      }
      if (e) store4(e + n0, v);
#pragma unroll
      for (int k = 0; k < 4; ++k) part = fmaf(v[k].x, v[k].x, fmaf(v[k].y, v[k].y, part));
    } else {
      for (int64_t n = n0; n < n0 + 4 && n < m.len; ++n) {
        float2 v = mp_value(u, a, n, 4, 4);
        v = make_float2(v.x - x[n].x, v.y - x[n].y);
        if (e) e[n] = v;
        part = fmaf(v.x, v.x, fmaf(v.y, v.y, part));
      }
    }
    sum += (double)part;
  }
  block_sum(sum, ws, m.partial);
}

// Samples left in t's row from t on (1 for the row's last), 0 past the batch.
__device__ __forceinline__ int64_t row_left(int64_t t, int64_t len, int64_t total) {
  if (t >= total) return 0;
  const int64_t row = total >> 32 ? t / len : (int64_t)((uint32_t)t / (uint32_t)len);
  return len - (t - row * len);
}

// Sample-wise forms: the batch's samples in one sequence, U per thread and 256
// apart.
template <bool FOUR, int U>
__global__ __launch_bounds__(256) void k_mp_loss_any(MpArgs m) {
  __shared__ double ws[4];
  const cfloat2p a = as_const(m.a);
  const int K = FOUR ? 4 : m.K, Q = FOUR ? 4 : m.Q;
  const int64_t total = m.S * m.len;
  double sum = 0.0;
  for (int64_t t0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x; t0 < total; t0 += (int64_t)gridDim.x * (256 * U)) {
    int64_t n[U];                                        // the sample's place in its row, -1 past the batch
    float2 v[U], w[U], P[U], D[U];
    float p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t left = row_left(t0 + 256 * u, m.len, total);
      n[u] = left ? m.len - left : -1;
      v[u] = make_float2(0.f, 0.f);
      if (left) {                                        // from -x on: e is often much smaller than v
        const float2 xv = m.x[t0 + 256 * u];
        v[u] = make_float2(-xv.x, -xv.y);
      }
    }
    for (int q = 0; q < Q; ++q) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w[u] = q <= n[u] ? m.u[t0 + 256 * u - q] : make_float2(0.f, 0.f);
        p[u] = norm2(w[u]);
      }
      tap_polys<false, U>(a, K, Q, q, p, P, D);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q <= n[u]) add_product(v[u], w[u], P[u]);
    }
    float part = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = t0 + 256 * u;
      if (n[u] < 0) continue;
      if (m.out) m.out[t] = v[u];
      part = fmaf(v[u].x, v[u].x, fmaf(v[u].y, v[u].y, part));
    }
    sum += (double)part;
  }
  block_sum(sum, ws, m.partial);
}

template <bool FOUR, int U>
__global__ __launch_bounds__(256) void k_mp_adj_any(MpArgs m) {
  const cfloat2p a = as_const(m.a);
  const int K = FOUR ? 4 : m.K, Q = FOUR ? 4 : m.Q;
  const float sc = m.scale ? 2.f * m.scale[0] : 1.f;
  const int64_t total = m.S * m.len;
  for (int64_t t0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x; t0 < total; t0 += (int64_t)gridDim.x * (256 * U)) {
    int64_t left[U];
    float2 uv[U], G[U], g[U], P[U], D[U];
    float p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      left[u] = row_left(t0 + 256 * u, m.len, total);
      uv[u] = left[u] ? m.u[t0 + 256 * u] : make_float2(0.f, 0.f);
      p[u] = norm2(uv[u]);
      G[u] = make_float2(0.f, 0.f);
    }
    for (int q = 0; q < Q; ++q) {
#pragma unroll
      for (int u = 0; u < U; ++u) g[u] = q < left[u] ? m.x[t0 + 256 * u + q] : make_float2(0.f, 0.f);
      tap_polys<true, U>(a, K, Q, q, p, P, D);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q < left[u]) add_adjoint(G[u], g[u], P[u], D[u], p[u], square(uv[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (left[u]) m.out[t0 + 256 * u] = make_float2(sc * G[u].x, sc * G[u].y);
  }
}

// The workgroups' sums in a fixed order.
__global__ __launch_bounds__(256) void k_mp_loss_sum(const double *partial, int n, float *loss) {
  __shared__ double ws[4];
  double sum = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) sum += partial[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) *loss = (float)(((ws[0] + ws[1]) + ws[2]) + ws[3]);
}

// Gu from u and the upstream gradient g, or (m.scale) 2 * scale[0] * g.
__global__ __launch_bounds__(256) void k_mp_adj(MpArgs m, int64_t runs, int64_t runs_per_row) {
  const cfloat2p a = as_const(m.a);
  const float sc = m.scale ? 2.f * m.scale[0] : 1.f;
  for (int64_t i = blockIdx.x; i < runs; i += gridDim.x) {
    const int64_t row = i / runs_per_row;
    const int64_t n0 = ((i - row * runs_per_row) * 256 + threadIdx.x) * 4;
    const float2 *u = m.u + row * m.len, *g = m.x + row * m.len;
    float2 *out = m.out + row * m.len;
    if (n0 + 8 <= m.len) {
      float2 uv[4], g0[4], g1[4], G[4], P, D;
      load4(u + n0, uv);
      load4(g + n0, g0);
      load4(g + n0 + 4, g1);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float p = norm2(uv[k]);
        const float2 u2 = square(uv[k]);
        G[k] = make_float2(0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          tap_poly<true>(a, 4, 4, q, p, P, D);
          add_adjoint(G[k], k + q < 4 ? g0[(k + q) & 3] : g1[(k + q) & 3], P, D, p, u2);
        }
        G[k] = make_float2(sc * G[k].x, sc * G[k].y);
      }
      store4(out + n0, G);
    } else {
      for (int64_t n = n0; n < n0 + 4 && n < m.len; ++n) {
        const float2 G = mp_adjoint(u[n], g, a, n, m.len, 4, 4);
        out[n] = make_float2(sc * G.x, sc * G.y);
      }
    }
  }
}

namespace {

struct MpGrid {
  int64_t runs, runs_per_row;
};

MpGrid mp_grid(const MpArgs &m) {
  const int64_t per_row = (m.len + 1023) / 1024;
  return {m.S * per_row, per_row};
}

// The runs form needs the model in use, rows that fill its workgroups, and
// enough of them to fill the chip (us of adjoint and loss, runs / sample-wise:
// 64 rows of 65536 19 24 / 23 27, 32 rows 11 15 / 14 17, 16 rows 7.6 11 / 7.4
// 11; 1024 of 4096 20 23 / 22 26, 3000 of 1000 18 21 / 18 21).
bool mp_runs(const MpArgs &m) {
  return m.K == 4 && m.Q == 4 && m.len >= 4096 && m.S * m.len >= (1 << 21);
}

unsigned mp_blocks(const MpArgs &m, int U, int64_t most) {
  return (unsigned)std::min<int64_t>((m.S * m.len + 256 * U - 1) / (256 * U), most);
}

}  // namespace

hipError_t launch_mp_loss(const MpArgs &m, float *loss, hipStream_t s) {
  int blocks = 0;
  if (m.S > 0 && m.len > 0) {
    const bool four = m.K == 4 && m.Q == 4;
    const int U = !four && m.S * m.len >= (1 << 19) ? 4 : 1;
    blocks = (int)mp_blocks(m, U, kMpLossBlocks);
    if (mp_runs(m)) {
      const MpGrid g = mp_grid(m);
      blocks = (int)std::min<int64_t>(g.runs, kMpLossBlocks);
      hipLaunchKernelGGL(k_mp_loss, dim3(blocks), dim3(256), 0, s, m, g.runs, g.runs_per_row);
    } else if (four) {
      hipLaunchKernelGGL((k_mp_loss_any<true, 1>), dim3(blocks), dim3(256), 0, s, m);
    } else if (U == 4) {
      hipLaunchKernelGGL((k_mp_loss_any<false, 4>), dim3(blocks), dim3(256), 0, s, m);
    } else {
      hipLaunchKernelGGL((k_mp_loss_any<false, 1>), dim3(blocks), dim3(256), 0, s, m);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_mp_loss_sum, dim3(1), dim3(256), 0, s, m.partial, blocks, loss);
  return hipGetLastError();
}

hipError_t launch_mp_adj(const MpArgs &m, hipStream_t s) {
  if (m.S <= 0 || m.len <= 0) return hipSuccess;
  const bool four = m.K == 4 && m.Q == 4;
  const int U = m.S * m.len >= (1 << 19) ? 2 : 1;
  const dim3 grid(mp_blocks(m, U, 1 << 20));
  if (mp_runs(m)) {
    const MpGrid g = mp_grid(m);
    const unsigned blocks = (unsigned)std::min<int64_t>(g.runs, 1 << 20);
    hipLaunchKernelGGL(k_mp_adj, dim3(blocks), dim3(256), 0, s, m, g.runs, g.runs_per_row);
  } else if (four) {
    if (U == 2) hipLaunchKernelGGL((k_mp_adj_any<true, 2>), grid, dim3(256), 0, s, m);
    else hipLaunchKernelGGL((k_mp_adj_any<true, 1>), grid, dim3(256), 0, s, m);
  } else {
    if (U == 2) hipLaunchKernelGGL((k_mp_adj_any<false, 2>), grid, dim3(256), 0, s, m);
    else hipLaunchKernelGGL((k_mp_adj_any<false, 1>), grid, dim3(256), 0, s, m);
  }
  return hipGetLastError();
}

}  // namespace dfh
