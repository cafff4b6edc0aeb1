// Host unit test of the rules that size a launch (csrc/host_logic.h): what
// they give stays inside the device's grid limits over the whole range of
// accepted sizes.
#include "host_logic.h"

#include <cstdio>
#include <cstdlib>
#include <initializer_list>

using namespace dfh::host;

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #c);    \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

// Motion: a grid row per firing, and one for the self-delay state.
static void motion() {
  for (int64_t w = 1; w <= 65536; w = w * 5 / 4 + 1)
    for (int64_t h = 1; h <= 65536; h = h * 5 / 4 + 1)
      for (int delay = 0; delay < 2; ++delay) {
        const int64_t bits = (w + 31) / 32 * h * 4, n = motion_chunk(bits, delay);
        CHECK(n >= 1 && n + delay <= 65535);
        CHECK(n == 1 || n * bits <= (512ll << 20));
      }
}

// One-launch scan: a workgroup per segment, a wavefront per branch.
static void scan_rows() {
  for (int B = 1; B <= 16; ++B)
    for (int64_t segs = 1; segs < 1ll << 34; segs = segs * 3 / 2 + 1)
      for (int64_t firings : {1, 64, 512, 513}) {
        const bool rows = scan_in_rows(segs, firings, B);
        CHECK(!rows || (firings <= 512 && segs * 64 * B < 1ll << 32));
        CHECK(rows || firings > 512 || segs * 64 * B > 1ll << 30);
      }
}

// Predistortion tiles: whole wavefronts, at most 256 threads, no larger than
// a firing needs; the caller's values stand; the matrix-core form keeps the
// shape it is fastest with.
static void tiles() {
  for (int64_t n : {1, 63, 64, 300, 4096})
    for (int64_t r = 1; r <= 1 << 17; r = r * 5 / 4 + 1)
      for (int mx = 0; mx < 2; ++mx)
        for (int tile : {0, 256, 512, 1024, 2048, 4096})
          for (int k : {0, 4, 8}) {
            const TileShape s = tile_shape(n, r, mx, tile, k);
            CHECK((s.K == 4 || s.K == 8) && s.tile % (64 * s.K) == 0 && s.tile >= 64 * s.K && s.tile <= 256 * s.K);
            CHECK(s.tile < r + 64 * s.K);
            CHECK((k == 0 || s.K == k) && (tile == 0 || s.tile <= tile || s.tile == 64 * s.K));
            if (mx && !tile && !k) CHECK(s.K == 4 && s.tile <= 1024);
          }
  CHECK(tile_shape(4096, 4096, false, 0, 0).tile == 2048 && tile_shape(4096, 4096, true, 0, 0).tile == 1024);
}

// Frame strips: four words only where the last strip has room for the word
// on its left, small batches of other widths never, large ones of large
// frames always, and never back to the other path as a batch grows.
static void strips() {
  for (int64_t W = 1; W <= 2000; ++W)
    for (int64_t H : {1, 16, 40, 251, 1080})
      for (int gauss = 0; gauss < 2; ++gauss) {
        const int few = strip_words(W, H, 1, gauss);
        CHECK(few == 4 || few == (W % 4 == 0 ? 1 : 0));
        CHECK(W % 16 != 0 || few == 4);
        bool four = false;
        for (int64_t n = 1; n <= 1ll << 34; n *= 4) {
          const int v = strip_words(W, H, n, gauss);
          CHECK(v == few || (v == 4 && W >= 20));
          CHECK(!four || v == 4);
          four = v == 4;
        }
        CHECK(four || W < 200 || H < 200);
      }
  CHECK(strip_words(854, 480, 64, true) == 4 && strip_words(854, 480, 64, false) == 4);
  CHECK(strip_words(333, 251, 4, true) == 0 && strip_words(20, 20, 1000, true) == 1);
}

// Launch shapes: each asked for once, however many there are.
static void shapes() {
  ShapeTable t;
  static char kernels[3];
  int made = 0;
  for (int pass = 0; pass < 2; ++pass)
    for (int k = 0; k < 3; ++k)
      for (int threads = 64; threads <= 256; threads += 64)
        for (size_t lds = 0; lds < 400; ++lds)
          for (int dev = 0; dev < 2; ++dev)
            CHECK(t.get(kernels + k, threads, lds, dev, [&] { return ++made, (int64_t)(k + threads + lds) * 2 + dev; }) ==
                  (int64_t)(k + threads + lds) * 2 + dev);
  CHECK(made == 3 * 4 * 400 * 2);
}

// Sample by sample: never for compiled taps with histories, always for one-sample rows,
// never for long firings in number; head rows hold the outputs.
static void samples() {
  for (int M = 1; M <= 32; ++M) {
    CHECK(head_lanes(M) >= M - 1 && (compiled_taps(M) == (M == 4 || M == 8 || M == 16)));
    for (int B = 1; B <= 16; ++B)
      for (DpdBatch k : {kRows, kTokens, kBatch}) {
        CHECK(!sample_wise(1 << 20, 4096, M, B, k));
        if (k == kRows) CHECK(sample_wise(1ll << 33, 1, M, B, k) && sample_wise(1, 1, M, B, k));
        else if (compiled_taps(M)) CHECK(!sample_wise(1 << 20, 1, M, B, k));
        if (M <= 2) CHECK(sample_wise(1ll << 30, 2, M, B, k));
      }
  }
}

int main() {
  samples();
  shapes();
  strips();
  tiles();
  motion();
  scan_rows();
  std::puts("launch rules: ok");
  return 0;
}
