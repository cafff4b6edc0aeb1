// Motion actor body: frame difference, threshold, 3x3 opening, per-frame
// changed count and data-dependent emission.
//
// Sec. 4.1 subtracts consecutive frames (the previous one arriving over a
// channel with a one-frame initial token) and thresholds against a constant.
// Per firing j:
//   m0 = |cur - prev| > thr
//   e  = AND of m0 over the in-frame 3x3 neighbourhood   (erosion)
//   o  = OR  of e  over the in-frame 3x3 neighbourhood   (dilation)
//   count_j = sum o;  emit_j = 1000*count_j >= permille*W*H
// Emission depends on the whole frame, so a batch runs
//   bits pass:   opened masks, bit-packed (32 pixels per word, transposed
//                bit order below), and counts
//   emit scan:   output slots of the emitted frames, channel indices
//   expand pass: emitted masks as 0/255 bytes at their output slots
//
// Bits pass layout: a wavefront owns a band of rows of one frame chunk and
// one chunk of 62 consecutive 32-pixel words (lane l <-> word chunk*62+l-1;
// lanes 0 and 63 are halo words).  It sweeps the rows of the band (plus two
// above and below) keeping, per frame, the last horizontal-AND rows and
// horizontal-OR rows in registers:
//   hm(y)   = m0(y) & left(m0(y)) & right(m0(y))  (neighbour pixels; edge
//             bits from the neighbour lanes)
//   e(y-1)  = hm(y-2) & hm(y-1) & hm(y)
//   he(y-1) = e(y-1) | left(e(y-1)) | right(e(y-1))
//   o(y-2)  = he(y-3) | he(y-2) | he(y-1)
// Outside the frame m0 counts as set (erosion ignores it) and e as clear
// (dilation ignores it).  Erosion and dilation over a square are separable,
// so this equals the 3x3 definitions exactly.  In the self-delay form a
// wavefront handles F consecutive frames per row, so each input row is
// loaded once for F frames (F+1 row loads per F outputs).
#include "common.h"

namespace dfh {

constexpr int MW_CHUNK = 62;   // output words per wavefront

typedef short i16x2 __attribute__((ext_vector_type(2)));

// Word of the neighbouring lane, one DPP move each (no LDS round trip):
// lane l receives lane l-1 (lane 0: 0) / lane l+1 (lane 63: 0).  Lanes 0
// and 63 are halo words whose results are discarded.
__device__ __forceinline__ uint32_t from_lower_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xF, 0xF, true);   // wave_shr:1
}
__device__ __forceinline__ uint32_t from_upper_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);   // wave_shl:1
}

// Mask words use a transposed bit order: pixel 4k + j of a word (dword k
// of its 32 bytes, byte j) is bit 8j + k.  The threshold's flags then
// gather with one byte permute and one shift-and-merge per dword, and the
// expand pass decodes a dword's four bytes with one mask and multiply.
__host__ __device__ constexpr int tbit(int x) { return 8 * (x & 3) + (x >> 2); }

// Natural-order mask (bit x = pixel x) to the transposed order.
__device__ __forceinline__ uint32_t to_tbits(uint32_t v) {
  uint32_t t = 0;
  for (int x = 0; x < 32; ++x) t |= ((v >> x) & 1u) << tbit(x);
  return t;
}

// Neighbour pixels in the transposed order: bit of pixel x receives pixel
// x+1 (right) or x-1 (left); across the word edge from the neighbouring
// lane's word (its pixel 0 is bit 0, its pixel 31 is bit 31).
__device__ __forceinline__ uint32_t tright(uint32_t m, uint32_t rw) {
  return (m >> 8) | ((m << 23) & 0x7F000000u) | (rw << 31);
}
__device__ __forceinline__ uint32_t tleft(uint32_t m, uint32_t lw) {
  return (m << 8) | ((m >> 23) & 0xFEu) | (lw >> 31);
}

// Even and odd bytes of a row's dwords spread into 16-bit lanes (byte
// permutes); in the self-delay form a frame's spread serves as the current
// frame of one output and the previous frame of the next.
struct Spread {
  i16x2 e[8], o[8];
};

__device__ __forceinline__ void spread(const uint32_t (&v)[8], Spread &s) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    s.e[k] = __builtin_bit_cast(i16x2, __builtin_amdgcn_perm(v[k], v[k], 0x0c020c00u));   // bytes 0, 2
    s.o[k] = __builtin_bit_cast(i16x2, __builtin_amdgcn_perm(v[k], v[k], 0x0c030c01u));   // bytes 1, 3
  }
}

// |cur - prev| > thr for the 32 pixels of a word (transposed order).  With
// d = cur - prev, a pixel is unchanged iff d - (thr+1) and -(thr+1) - d are
// both negative, i.e. bit 15 of their AND: pixels 0 and 2 of a dword in the
// even product's bits 15 and 31, pixels 1 and 3 in the odd one's.  One
// byte permute puts pixel j's flag in bit 7 of byte j, a shift by 7 - k and
// a mask move it to bit 8j + k; the word is inverted once.
__device__ __forceinline__ uint32_t thresh_tbits(const Spread &c, const Spread &p, i16x2 t1, i16x2 nt1) {
  uint32_t keep = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const i16x2 de = c.e[k] - p.e[k], dd = c.o[k] - p.o[k];
    const uint32_t ye = __builtin_bit_cast(uint32_t, de - t1) & __builtin_bit_cast(uint32_t, nt1 - de);
    const uint32_t yo = __builtin_bit_cast(uint32_t, dd - t1) & __builtin_bit_cast(uint32_t, nt1 - dd);
    const uint32_t g = __builtin_amdgcn_perm(yo, ye, 0x07030501u);   // ye.b1, yo.b1, ye.b3, yo.b3
    keep |= (g >> (7 - k)) & (0x01010101u << k);
  }
  return ~keep;
}

// 16 bytes at any byte address
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((aligned(1))) u32x4_any;

// One row of the F+1 frames a wavefront needs: fr[f] is the previous frame of
// frame f and fr[f+1] its current frame (self-delay form: frames j0-1 ..
// j0+F-1 of the input channel, the first from the state for j0 = 0; the
// two-channel form has F = 1: fr[0] from the PREV channel, fr[1] from CUR).
// Callers clamp y into the frame and point the frames past the batch at its
// last frame (those results are masked).  The wavefront's 64 words are the
// 2 KiB from byte xs of the row; it loads them as two contiguous KiB spans
// (lane l: 16 bytes at xs + 16 l and at xs + 1024 + 16 l; nothing outside the
// row) ...
// A row may start at any byte, and the last 16 bytes of a row may reach past
// its end: into the next row, or behind a channel's or state's last frame
// into the kFrameSlack bytes allocated there.  Those pixels are masked.
template <int F>
__device__ __forceinline__ void load_spans(const uint8_t *const (&fr)[F + 1], int y, int xs, int W,
                                           uint32_t (&raw)[F + 1][8]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int f = 0; f <= F; ++f)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int off = xs + 1024 * h + 16 * lane;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (off >= 0 && off < W)
        v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(fr[f] + (int64_t)y * W + off));
      raw[f][4 * h + 0] = v.x;
      raw[f][4 * h + 1] = v.y;
      raw[f][4 * h + 2] = v.z;
      raw[f][4 * h + 3] = v.w;
    }
}

// ... and passes them through LDS (stg: (F+1) x 512 words of this
// wavefront), so that each lane ends with its own 32 bytes (bytes 32 l ..
// 32 l + 31 of the span) in buf.
template <int F>
__device__ __forceinline__ void stage_spans(uint32_t *stg, const uint32_t (&raw)[F + 1][8], uint32_t (&buf)[F + 1][8]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int f = 0; f <= F; ++f)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      *reinterpret_cast<u32x4 *>(stg + 512 * f + 256 * h + 4 * lane) =
          u32x4{raw[f][4 * h], raw[f][4 * h + 1], raw[f][4 * h + 2], raw[f][4 * h + 3]};
#pragma unroll
  for (int f = 0; f <= F; ++f)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + 512 * f + 8 * lane + 4 * h);
      buf[f][4 * h + 0] = v.x;
      buf[f][4 * h + 1] = v.y;
      buf[f][4 * h + 2] = v.z;
      buf[f][4 * h + 3] = v.w;
    }
}

// Work items in XCD-contiguous order: workgroups are dispatched to the 8
// XCDs round robin (workgroup b to XCD b % 8), so item k runs on XCD
// k / per_xcd, and the items an XCD runs in turn are consecutive: the bands
// of a frame group and the next frame groups.  A band's halo rows and the
// previous frame a frame group re-reads are then loaded by workgroups of one
// XCD at about the same time, and come from its L2.  Returns -1 for the
// padding workgroups of a grid rounded up to a multiple of 8.
__device__ __forceinline__ int xcd_item(int b, int n_items) {
  const int per_xcd = (n_items + 7) >> 3;
  const int k = (b & 7) * per_xcd + (b >> 3);
  return k < n_items ? k : -1;
}

template <int F>
__global__ __launch_bounds__(64) void k_motion_bits(MotionArgs a, int rows, int n_bands, int n_chunks, int n_items) {
  const int lane = threadIdx.x;
  const int blk = xcd_item(blockIdx.x, n_items);
  if (blk < 0) return;
  const int chunk = blk % n_chunks;
  const int band = (blk / n_chunks) % n_bands;
  const int64_t j0 = (int64_t)(blk / (n_chunks * n_bands)) * F;
  const int nfr = (int)min((int64_t)F, a.n - j0);
  const int H = a.H, W = a.W, wpr = a.words_per_row;
  const int c = chunk * MW_CHUNK + lane - 1;
  const bool word_in = c >= 0 && c < wpr;
  const bool out_lane = lane >= 1 && lane <= MW_CHUNK && word_in;
  const uint32_t valid = (c == wpr - 1 && (W & 31)) ? to_tbits((1u << (W & 31)) - 1u) : 0xFFFFFFFFu;
  const int64_t wh = (int64_t)W * H;
  const short t1s = (short)(a.thr + 1);
  const i16x2 t1 = {t1s, t1s}, nt1 = {(short)-t1s, (short)-t1s};
  const int y0 = band * rows, y1 = min(H, y0 + rows);
  uint32_t *__restrict__ bits = a.bits;

  // frame base pointers of the chunk (see load_spans)
  const uint8_t *fr[F + 1];
  {
    const int64_t Rc = a.cur_idx[0];
#pragma unroll
    for (int f = 0; f <= F; ++f) {
      if (a.prev) {
        fr[f] = f == 0 ? a.prev + ((a.prev_idx[0] + j0) & a.prev_mask) * wh : a.cur + ((Rc + j0) & a.cur_mask) * wh;
      } else {
        const int64_t j = j0 + min(f, nfr) - 1;            // past the batch: its last frame
        fr[f] = j < 0 ? a.state : a.cur + ((Rc + j) & a.cur_mask) * wh;
      }
    }
  }

  uint32_t hm2[F], hm1[F], he3[F], he2[F];
  int cnt[F];
#pragma unroll
  for (int f = 0; f < F; ++f) hm2[f] = hm1[f] = he3[f] = he2[f] = 0, cnt[f] = 0;

  auto process = [&](const uint32_t (&buf)[F + 1][8], int y) {
    const bool in = y >= 0 && y < H && word_in;
    const bool e_in = y - 1 >= 0 && y - 1 < H && word_in;
    Spread sp, sc;
    spread(buf[0], sp);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      if (f >= nfr) break;                                  // uniform
      spread(buf[f + 1], sc);
      const uint32_t th = thresh_tbits(sc, sp, t1, nt1);
      sp = sc;
      const uint32_t m0 = in ? (th | ~valid) : 0xFFFFFFFFu; // outside the frame: set
      // horizontal AND with the neighbour words' edge bits
      const uint32_t lw = from_lower_lane(m0), rw = from_upper_lane(m0);
      const uint32_t hm = m0 & tleft(m0, lw) & tright(m0, rw);
      const uint32_t e = e_in ? (hm2[f] & hm1[f] & hm & valid) : 0u;   // e(y-1); outside: clear
      const uint32_t le = from_lower_lane(e), re = from_upper_lane(e);
      const uint32_t he = e | tleft(e, le) | tright(e, re);
      const uint32_t o = (he3[f] | he2[f] | he) & valid;    // o(y-2)
      const int yo = y - 2;
      if (yo >= y0 && yo < y1 && out_lane) {
        cnt[f] += __popc(o);
        bits[(j0 + f) * (int64_t)H * wpr + (int64_t)yo * wpr + c] = o;
      }
      hm2[f] = hm1[f];
      hm1[f] = hm;
      he3[f] = he2[f];
      he2[f] = he;
    }
  };

  uint32_t A[F + 1][8], Bf[F + 1][8];
#pragma unroll
  for (int f = 0; f <= F; ++f)
#pragma unroll
    for (int k = 0; k < 8; ++k) A[f][k] = Bf[f][k] = 0;
  const int ylast = y1 + 1;
  // the next row's loads are in flight (raw) while the current row, already
  // staged through LDS, is processed
  __shared__ uint32_t stg[F + 1][512];
  const int xs = (chunk * MW_CHUNK - 1) * 32;
  auto clampy = [&](int y) { return min(max(y, 0), H - 1); };
  load_spans<F>(fr, clampy(y0 - 2), xs, W, Bf);
  stage_spans<F>(&stg[0][0], Bf, A);
  for (int y = y0 - 2; y <= ylast; ++y) {
    if (y + 1 <= ylast) load_spans<F>(fr, clampy(y + 1), xs, W, Bf);
    process(A, y);
    if (y + 1 > ylast) break;
    stage_spans<F>(&stg[0][0], Bf, A);
  }
#pragma unroll
  for (int f = 0; f < F; ++f) {
    int t = cnt[f];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
    if (lane == 0 && f < nfr && t) atomicAdd(&a.count[j0 + f], t);
  }
}

// Expand the bit-packed mask of every emitted frame to 0/255 bytes at the
// frame's output slot.  One thread per 16-pixel half word, so the lanes of a
// wavefront store one contiguous 1 KiB span per instruction.
// The same pass leaves the batch's counts at zero for the next batch (the
// emit scan has read them) and, with state_src set, copies the batch's last
// frame to the self-delay state (grid row n: 16 bytes per thread, the last
// ones into the slack; nothing in this pass reads the frames or the state).
__global__ __launch_bounds__(256) void k_motion_expand(MotionArgs a) {
  const int64_t j = blockIdx.y;
  const int W = a.W, H = a.H, wpr = a.words_per_row;
  const int64_t wh = (int64_t)W * H;
  const int64_t hw = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j == a.n) {
    if (hw * 16 < wh) {
      const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(a.state_src + hw * 16));
      *reinterpret_cast<u32x4 *>(a.state + hw * 16) = v;
    }
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.count[j] = 0;
  const int64_t slot = a.emit_off[j];
  if (slot < 0) return;                                 // uniform: not emitted
  const int64_t *base = a.emit_off + a.n + 1;           // write positions before the batch (masks, indices)
  if (blockIdx.x == 0 && threadIdx.x == 0) a.index_out[(base[1] + slot) & a.index_mask] = a.frame_base + j;
  if (hw >= 2 * (int64_t)H * wpr) return;
  const int64_t wi = hw >> 1;
  const int half = (int)(hw & 1);
  const int y = (int)(wi / wpr), c = (int)(wi - (int64_t)y * wpr);
  const uint32_t o = a.bits[j * (int64_t)H * wpr + wi] >> (4 * half);
  const int x = c * 32 + 16 * half;
  uint8_t *dst = a.out + ((base[0] + slot) & a.out_mask) * wh + (int64_t)y * W + x;
  uint32_t v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = ((o >> k) & 0x01010101u) * 0xFFu;   // dword k: pixel 4k + j <- bit 8j + k
  if (x + 16 <= W) {
    const u32x4 val = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(val, reinterpret_cast<u32x4_any *>(dst));
  } else {
    for (int i = 0; i < W - x; ++i) dst[i] = (uint8_t)(v[i >> 2] >> (8 * (i & 3)));
  }
}

// Exclusive scan of emit flags and batch commit: emit_off[j] = output slot of
// firing j or -1, emit_off[n] = number of emitted frames, emit_off[n+1..n+2] =
// write positions of the mask and index channels before the batch (the expand
// pass, the batch's last, places its tokens from them); then every channel
// counter advances, and the new write positions go to host memory too, so that
// the host learns them without a copy.  One wavefront, ballot-based.
__global__ __launch_bounds__(64) void k_emit_commit(MotionCommitArgs a) {
  const int lane = threadIdx.x;
  const uint64_t below_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
  int64_t carry = 0;
  for (int64_t c = 0; c < a.n; c += 64) {
    const int64_t j = c + lane;
    const bool f = j < a.n && 1000 * (int64_t)a.count[j] >= a.thresh;
    const uint64_t bal = __ballot(f);
    if (j < a.n) a.emit_off[j] = f ? carry + __popcll(bal & below_mask) : -1;
    carry += __popcll(bal);
  }
  if (lane != 0) return;
  const int64_t out0 = a.out_idx[1], index0 = a.index_idx[1];
  a.emit_off[a.n] = carry;
  a.emit_off[a.n + 1] = out0;
  a.emit_off[a.n + 2] = index0;
  a.cur_idx[0] += a.n;
  if (a.prev_idx) a.prev_idx[0] += a.n;
  a.out_idx[1] = out0 + carry;
  a.index_idx[1] = index0 + carry;
  check_chan(a.cur_idx, a.err);
  if (a.prev_idx) check_chan(a.prev_idx, a.err);
  check_chan(a.out_idx, a.err);
  check_chan(a.index_idx, a.err);
  if (!a.host) return;
  const uint64_t seq = (uint64_t)a.seq << 32;
  __hip_atomic_store(&a.host->word[0], seq | (uint32_t)(out0 + carry), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&a.host->word[1], seq | (uint32_t)(index0 + carry), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int F>
static hipError_t launch_bits(const MotionArgs &a, hipStream_t s, int64_t items, int rows, int n_bands,
                              int n_chunks) {
  if (items > 0x7ffffff0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((items + 7) / 8 * 8));
  hipLaunchKernelGGL(k_motion_bits<F>, grid, dim3(64), 0, s, a, rows, n_bands, n_chunks, (int)items);
  return hipGetLastError();
}

// Shape of the bits pass: F frames per wavefront in the self-delay form (F + 1
// row loads per F frames; the two-channel form has F = 1) and bands of `rows`
// rows (4 rows more are loaded than written).  Large F and bands read less,
// but a wavefront walks its rows one after the other, so a batch that leaves
// the 1024 SIMDs short of wavefronts wants smaller ones: the largest F with
// 32-row bands that still gives 120000 word columns (2000 wavefronts of 60
// words), else F = 1 and 16, 8 or 4 rows.  Batch body in us by F/rows:
//   1920x1080  300 frames  4/32 292  2/32 313  1/32 369  4/16 312
//              120         4/32 161  2/32 136  1/32 148  4/16 140
//               30         4/32  92  2/32  65  1/16  54  1/8 56
//                8         4/32  81  1/16  33  1/8   31  1/4 37
//                1         4/32  43  1/8   20  1/4   18
//    640x480    64         4/32  81  1/16  41  1/8   37  1/4 44
//    320x240   256         4/32  87  1/32  61  1/16  48  1/8 51
//               24         4/32  82  1/16  26  1/8   23  1/4 24
//   3840x2160   20         4/32 125  2/32 111  1/32 113  1/16 126
struct BitsShape {
  int F, rows;
};

static BitsShape bits_shape(const MotionArgs &a, int n_chunks) {
  const auto waves = [&](int F, int rows) {
    return (int64_t)n_chunks * ((a.H + rows - 1) / rows) * ((a.n + F - 1) / F);
  };
  const int64_t words = a.words_per_row < MW_CHUNK ? a.words_per_row : MW_CHUNK;
  for (int F = a.prev ? 1 : 4; F >= 1; F /= 2)
    if (waves(F, 32) * words >= 120000) return {F, 32};
  if (waves(1, 16) >= 2000) return {1, 16};
  return {1, waves(1, 8) >= 500 ? 8 : 4};
}

hipError_t launch_motion_count(const MotionArgs &a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (a.n + (a.state_src ? 1 : 0) > 65535) return hipErrorInvalidValue;   // grid rows of the expand pass
  const int n_chunks = (a.words_per_row + MW_CHUNK - 1) / MW_CHUNK;
  const BitsShape sh = bits_shape(a, n_chunks);
  const int n_bands = (a.H + sh.rows - 1) / sh.rows;
  const int64_t items = (int64_t)n_chunks * n_bands * ((a.n + sh.F - 1) / sh.F);
  if (sh.F == 4) return launch_bits<4>(a, s, items, sh.rows, n_bands, n_chunks);
  if (sh.F == 2) return launch_bits<2>(a, s, items, sh.rows, n_bands, n_chunks);
  return launch_bits<1>(a, s, items, sh.rows, n_bands, n_chunks);
}

hipError_t launch_motion_emit_commit(const MotionCommitArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_emit_commit, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_motion_emit(const MotionArgs &a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  const int64_t halves = 2 * (int64_t)a.H * a.words_per_row;
  // grid row n copies the state: 16 bytes per thread cover the frame
  // (halves * 16 >= W * H)
  dim3 grid((unsigned)((halves + 255) / 256), (unsigned)(a.n + (a.state_src ? 1 : 0)));
  hipLaunchKernelGGL(k_motion_expand, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace dfh
