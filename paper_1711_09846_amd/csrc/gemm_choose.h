// Which tile a population-batched product takes, and which weight gradients are formed in pieces: rules on sizes alone.
#pragma once
#include <cstdint>

namespace pbt {

struct TileShape { int bm, bn; };
inline int64_t tile_count(int M, int N, int batch, int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch; }

constexpr int64_t GL_MAX_PITCH = 1 << 24;      // elements per row below which every offset inside a slab of 64 rows stays under it

enum GlShape { GL_256 = 0, GL_128, GL_128x64, GL_64 };
inline TileShape gl_shape(GlShape t) { return t == GL_256 ? TileShape{256, 256} : t == GL_128 ? TileShape{128, 128} : t == GL_128x64 ? TileShape{128, 64} : TileShape{64, 64}; }
inline int gl_upper_tiles(int N, TileShape t) {
  const int tiles = (N + t.bm - 1) / t.bm;
  return tiles * (tiles + 1) / 2;
}

// The shape with the shortest estimate (us, to *estimate), from what tiles take on this card (us, about 2 GHz, where the matrix pipes leave it): a compute unit's first tile LATENCY per 64
// of K, each further one RATE; FIXED per tile for its first loads and a plain epilogue, HEAVY more for a long one (an exponential, a Philox block or
// another array per element).  Fitted to 60 shapes of all three layouts; the shape it picks is 0.3 % slower than the best one on average, 7 % at most.  At its
// lines: 16 members' 4096 x 2048 x 512 take 256x256 tiles with a plain epilogue (150 us; 128x128: 192) and 128x128 with dropout (283; 300), 64 members' 2048 x 1024
// with GELU 128x128 at K = 256 (188; 196) and 256x256 at K = 1024 (380; 440); 6 members' 720 x 192 x 776 take 64x64 (7.9 us; 128x64: 9.7) and 720 x 776 x 192
// 128x64 (6.6; 64x64: 8.2); one product 1536 x 1536 x 4096 64x64 (43.9; 128x128: 59.5).
// Rows so long that 256 of them exceed a buffer offset take the 64-row tile (and have no estimate).
// square: RBF sums, whose tiles are square and whose long epilogue has a slower path for tiles on the diagonal of a symmetric product (upper) and at a ragged
// edge: GENERAL more for each of those that a compute unit gets.  Held-out passes of 6 members, 1500 rows of 256, with the tiles counted as if all
// of a symmetric product were formed: 97.4 us, 82.7 now; 16 members, 1024 rows of 256: 93.1, 83.5; 8 members, 1024 rows of 64: 52.7, 48.3.
inline GlShape gl_choose(int M, int N, int K, int batch, bool heavy, bool square, int64_t pitch, bool upper = false,
                         double* estimate = nullptr) {
  if (pitch >= GL_MAX_PITCH / 4) return GL_64;
  constexpr double LATENCY[4] = {1.9, 1.09, 0.38, 0.255}, RATE[4] = {1.9, 0.5, 0.42, 0.21}, FIXED[4] = {3.4, 0.97, 0.75, 0.63}, HEAVY[4] = {14.5, 3.0, 4.0, 0.5};
  constexpr double RBF[4] = {14.5, 3.0, 0.0, 0.8}, GENERAL[4] = {6.0, 3.0, 0.0, 0.5};
  GlShape best = GL_256;
  double least = 0.;
  for (int t = GL_256; t <= GL_64; ++t) {
    const TileShape sh = gl_shape((GlShape)t);
    if (square && sh.bm != sh.bn) continue;
    const int64_t tiles_m = (M + sh.bm - 1) / sh.bm, tiles_n = (N + sh.bn - 1) / sh.bn;
    const int64_t per_cu = ((upper ? gl_upper_tiles(N, sh) : tiles_m * tiles_n) * batch + 255) / 256;
    const double slabs = K / 64., fixed = FIXED[t] + (square ? RBF[t] : heavy ? HEAVY[t] : 0.);
    double cost = slabs * LATENCY[t] + fixed + (double)(per_cu - 1) * (slabs * RATE[t] + fixed);
    if (square) {
      const int64_t general = (upper ? tiles_n : 0) + (N % sh.bn ? tiles_m : 0) + (!upper && M % sh.bm ? tiles_n : 0);
      cost += GENERAL[t] * (double)((general * batch + 255) / 256);
    }
    if (t == GL_256 || cost < least) {
      least = cost;
      best = (GlShape)t;
    }
  }
  if (estimate) *estimate = least;
  return best;
}

// A weight gradient's product is over a member's rows, a long contraction: where a population's tiles are few each is a serial chain of slabs on one of a few
// compute units.  Cut into WGRAD_PARTS pieces it is as many products of a quarter of the rows, whose results are added up in order afterwards.
constexpr int WGRAD_PARTS = 4;
// A matrix of at most 64 256 x 256 tiles over at least 4096 rows: a piece keeps the large tile that the whole cannot give to every compute unit, a
// closer call than the estimates can make (per step: one member, d_model 512, d_ff 2048, 4096 rows 807 us by the estimates alone, 731 so; eight members,
// 256 and 1024: 1493, 1445).  Working memory is kept for these pieces.
inline bool wgrad_large_pieces(int P, int rows, int K, int N) {
  if (N % 4 || ((int64_t)K * N) % 4) return false;
  return tile_count(K, N, P, 256, 256) <= 64 && K >= 256 && N >= 256 && rows % (WGRAD_PARTS * 64) == 0 && rows / WGRAD_PARTS >= 1024;
}
// Those, and where the estimates of whole and pieces (3 us more, and the traffic of adding them up) say so, if the pieces fit memory that is there anyway: one member,
// 192 and 776, 4096 rows: 708 us whole, 504 in pieces; six members, 96 and 384: 891, 713; one member, 128 and 512, 8192 rows: 1115, 679.  Six
// members' 192 x 776 from 720 rows stay whole (10.2 us; 12.3 + 4.6 in pieces).
inline bool wgrad_in_parts(int P, int rows, int K, int N) {
  if (wgrad_large_pieces(P, rows, K, N)) return true;
  if (N % 4 || ((int64_t)K * N) % 4 || rows % WGRAD_PARTS) return false;
  double whole = 0., pieces = 0.;
  const int64_t pitch = K > N ? K : N;
  gl_choose(K, N, rows, P, false, false, pitch, false, &whole);
  gl_choose(K, N, rows / WGRAD_PARTS, P * WGRAD_PARTS, false, false, pitch, false, &pieces);
  return pieces + 3.0 + (double)P * K * N * 4 * (WGRAD_PARTS + 1) / 5e6 < whole;
}

}  // namespace pbt
