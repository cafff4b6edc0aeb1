// Host-side arithmetic of the runtime that involves no device: channel slot
// maps and the runs of consecutive slots a host copy covers, the slot-0 copy
// of the paper's delay-token layout, and the batch whose ring slots a
// streamed write reuses.  Plain C++ (no HIP), so that a host unit test can
// build it under AddressSanitizer / UndefinedBehaviorSanitizer.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <new>
#include <tuple>

namespace dfh {
namespace host {

inline int64_t next_pow2(int64_t v) {
  int64_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

// A channel's slots: a ring of `cap` (a power of two) slots, or the paper's
// layout of Sec. 3.2 with period P (2r, or 3r with one delay token: 3r + 1
// slots, writes filling slots 1..3r in turn, reads taking 0..3r-1).
struct SlotMap {
  int64_t cap = 0;      // ring capacity (period == 0)
  int64_t period = 0;   // paper layout period, 0 for a ring
  bool delay = false;   // paper layout with its one delay token
};

inline int64_t read_slot(const SlotMap &m, int64_t p) { return m.period ? p % m.period : (p & (m.cap - 1)); }

inline int64_t write_slot(const SlotMap &m, int64_t p) {
  if (!m.period) return p & (m.cap - 1);
  return m.delay ? 1 + (p - 1) % m.period : p % m.period;
}

// Exclusive end of the slots one run of a host copy may cover before the
// access pattern wraps to its first slot.
inline int64_t run_end(const SlotMap &m, bool to_ring) {
  if (!m.period) return m.cap;
  return (to_ring && m.delay) ? m.period + 1 : m.period;
}

// The next run of a copy of tokens [q, q + left): its first slot and length.
struct Run {
  int64_t slot, count;
};
inline Run next_run(const SlotMap &m, int64_t q, int64_t left, bool to_ring) {
  const int64_t slot = to_ring ? write_slot(m, q) : read_slot(m, q);
  const int64_t room = run_end(m, to_ring) - slot;
  return Run{slot, left < room ? left : room};
}

// Delay-token layout: the position in [pos, pos + n) whose write fills slot
// P (so that slot P must then be copied to slot 0), or -1.  Position 0 is the
// delay token itself and is never written.  With n <= P (what admission
// allows) there is at most one.
inline int64_t fixup_position(int64_t pos, int64_t n, int64_t P) {
  if (n <= 0 || P <= 0) return -1;
  const int64_t first = pos + ((P - (pos % P)) % P);   // first multiple of P at or after pos
  return (first < pos + n && first != 0) ? first : -1;
}

// Streamed writes: batches of n tokens start at `base`, n apart; a write
// whose last position is `last` reuses the ring slots of the batch holding
// position last - cap, if that position belongs to a batch.
inline int64_t reused_batch(int64_t last, int64_t cap, int64_t base, int64_t n) {
  const int64_t p = last - cap;
  return p < base ? -1 : (p - base) / n;
}

// Firings of a motion batch one launch may cover: its passes have a grid row
// per firing, at most 65535, and with a self-delay the last pass one more for
// the state; and at most 512 MiB of staged mask bits.
inline int64_t motion_chunk(int64_t frame_bits, bool self_delay) {
  const int64_t rows = 65535 - (self_delay ? 1 : 0), staged = (512ll << 20) / frame_bits;
  return staged < 1 ? 1 : staged < rows ? staged : rows;
}

// A launch has fewer than 2^32 threads; half of that is the most asked for.
constexpr int64_t kMaxThreads = 1ll << 31;

// Segments short enough for the one-launch scan (a wavefront per branch walks
// a segment 64 firings at a time), and few enough for its grid.
constexpr int64_t kRowFirings = 512;
inline bool scan_in_rows(int64_t n_segs, int64_t seg_firings, int B_max) {
  return seg_firings <= kRowFirings && n_segs <= kMaxThreads / (64 * B_max);
}

// Shape of a predistortion tile: outputs per thread and per workgroup (at
// most 256 threads).  A caller's own choice of either value stands.
// By default 2048 outputs with eight per thread where firings fill such tiles
// and there is one for each of the 256 compute units (fewer scalar loads, LDS
// reads and |x|^2 per output; ms against 1024 with four: 32 firings of 65536,
// 10 taps 0.022 / 0.029; 256 of 4096, 16 taps 0.016 / 0.021; 4096 of 4096
// 0.108 / 0.107; 128 of 4096 0.014 / 0.014), else 1024 with four (777 firings
// of 1000: 0.019 / 0.023).  The matrix-core form (mx) keeps 1024 with four:
// its row sums make a 2048-output tile 88 KB of LDS, one workgroup a compute
// unit (us a pass, 2048/8 and 1024/4: 4096 firings of 4096 361 / 281, 256 of
// 4096 48 / 47, 32 of 65536 66 / 59).
// The tile is a multiple of 64*K outputs and no larger than needed for one
// firing.
struct TileShape {
  int K, tile;
};
inline TileShape tile_shape(int64_t n_firings, int64_t r, bool mx, int tile, int outputs_per_thread) {
  const bool big = !mx && tile <= 0 && r >= 2048 && n_firings * r >= 256 * 2048;
  const int K = outputs_per_thread == 8 || (outputs_per_thread == 0 && big) ? 8 : 4;
  int tl = tile > 0 ? tile : (outputs_per_thread == 0 && big ? 2048 : 1024);
  const int64_t rr = ((r + 64 * K - 1) / (64 * K)) * (64 * K);
  if ((int64_t)tl > rr) tl = (int)rr;
  tl = (tl / (64 * K)) * (64 * K);
  if (tl < 64 * K) tl = 64 * K;
  if (tl / K > 256) tl = 256 * K;
  return TileShape{K, tl};
}

// Frame actors: words per strip of the word path (4 or 1), or 0 for the byte
// path, by frame size, batch and actor (Gauss, else Med).  A strip of four
// words is a wavefront's lane and walks kStripRows rows one after the other:
// 12 us however little there is (one word 8, bytes 4), 3.7 ns more per
// wavefront, idle lanes included, but least per pixel where the wavefronts are
// full.  Bytes take 1.15 ns per 256 pixels (Gauss; Med 0.55).  us of Gauss and
// Med, four words / the other path:
//   width not a multiple of 4, bytes:
//     333x251  6 frames 14 14 /  6  5    24  13 13 / 13  7    120   15 16 / 48 25
//     65x48  481        17 16 / 11  7   962  13 14 / 19 11   3205   26 23 / 51 30
//     33x17 1783        18 17 /  9  5  17825 79 80 / 52 29
//   a multiple of 4, one word:
//     1000x600 17       15 19 / 12 13    33  17 20 / 19 17     67   29 24 / 38 29
//     100x75 1333       20 19 / 17  9  13333 191 112 / 195 93
//     20x20 25000      105 106 / 47 42
// Multiples of 16 take four words at any size.
constexpr int kStripRows = 16;

inline int64_t strip_lanes(int64_t W, int64_t H, int V) {
  return (H + kStripRows - 1) / kStripRows * ((W + 4 * V - 1) / (4 * V));
}

inline int strip_words(int64_t W, int64_t H, int64_t n_frames, bool gauss) {
  if (W % 16 == 0) return 4;
  const int other = W % 4 == 0 ? 1 : 0;
  if (W < 20) return other;                  // no room for the word left of the last strip
  const int64_t lanes = strip_lanes(W, H, 4), waves = (lanes + 63) / 64;
  if (other) {
    const bool full = 4 * lanes >= 3 * 64 * waves;
    return full && n_frames * W * H >= (gauss ? 20000000 : 32000000) ? 4 : 1;
  }
  const int64_t blocks = (W * H + 255) / 256;
  return n_frames * blocks * (gauss ? 1150 : 550) > 8500000 + n_frames * waves * 3700 ? 4 : 0;   // picoseconds
}

// Lanes of a firing's row in the head pass: 16 for the compiled tap counts (4,
// 8, 16), else the fewest that hold the M - 1 outputs.
inline bool compiled_taps(int M) { return M == 4 || M == 8 || M == 16; }
inline int head_lanes(int M) { return compiled_taps(M) || (M > 9 && M <= 17) ? 16 : M <= 5 ? 4 : M <= 9 ? 8 : 32; }

// Whether a batch of n firings (or rows) of r samples runs sample by sample
// (k_dpd_samples) and not in tiles: rows without histories with any taps, the
// rest where the taps are not compiled in (a compiled head pass adds its terms
// in another form).
// A tile costs 0.45 ns and 14.5 ps per coefficient however few of its 256
// outputs a short firing fills, and firings with histories cost the head pass
// 70 ps a lane (110 with the tables).  A sample costs 2 ps (6 with histories)
// and 0.24 per coefficient, and where firings have histories its share of the
// wavefront's corrections, 0.055 per term, of which one thread forms all of its
// own (12 ns a term).  us of a call, samples / tiles:
//   rows without control tokens, 10 branches of 12 taps: 100 of 16 20 / 26,
//     30000 of 16 26 / 80, of 64 68 / 78, of 96 96 / 77; 100000 of 16 with 16
//     taps 66 / 266
//   rows of 100 firings, in all 30000 of 3 branches and 3 taps: of 8 26 / 33, of
//     64 34 / 35, of 96 42 / 35; 200000 of 8 with 10 and 9 180 / 312
//   a batch of 30000 with 3 and 3: of 2 42 / 60, of 48 67 / 67, of 96 88 / 73;
//     with 6 and 12: of 16 94 / 113, of 32 134 / 116; 200000 of 16 408 / 592
enum DpdBatch { kRows, kTokens, kBatch };    // stateless without and with control tokens, an actor's batch
inline bool sample_wise(int64_t n, int64_t r, int M, int B, DpdBatch kind) {
  if (compiled_taps(M) && kind != kRows) return false;
  const int64_t N = n * r, tiles = n * ((r + 255) / 256), terms = (M - 1) * B * (B + 19) / 2;   // picoseconds below
  if (kind == kRows) return N / 1000 * (2000 + 240 * M * B) < 6000000 + tiles * (450 + 29 * M * B / 2);
  const int64_t each = 6000 + 240 * M * B + 55 * terms, tile = 450 + 29 * M * (B + 1) / 4;
  if (kind == kTokens)
    return 12000 * terms + N / 1000 * (each * 27 / 20) < 8000000 + tiles * tile + n * 70 * head_lanes(M);
  return 12000 * terms + N / 1000 * (each * 11 / 10) + n * 120 + 5000000 < tiles * tile + n * 110 * head_lanes(M);
}

// Numbers known per launch shape (kernel, threads, LDS bytes, device), for any
// number of shapes (a program has as many as its actors' tap counts, branch
// counts and tiles make), from any thread.
class ShapeTable {
 public:
  // The shape's number; made by `make` when it is not known yet.
  template <class Make>
  int64_t get(const void *kernel, int threads, size_t lds_bytes, int device, Make make) {
    std::lock_guard<std::mutex> lock(mu_);
    const Key k{kernel, threads, lds_bytes, device};
    const auto it = known_.find(k);
    if (it != known_.end()) return it->second;
    const int64_t n = make();
    try {
      known_[k] = n;
    } catch (const std::bad_alloc &) {                   // not kept
    }
    return n;
  }

 private:
  typedef std::tuple<const void *, int, size_t, int> Key;
  std::mutex mu_;
  std::map<Key, int64_t> known_;
};

}  // namespace host
}  // namespace dfh
