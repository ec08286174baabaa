// Choice of the bf16 GEMM tile.  Plain host code, without HIP, so that the tests
// can ask which tiles their shapes reach.
#pragma once

namespace cs {

enum Bf16Tile {
  W4_256x256, W4_224x256, W4_192x256, W4_160x256, W4_128x128, W4_64x64,
  RING_128x128, RING_64x128, RING_64x64, RING_32x64, RING_32x32, N_TILES
};

// Time of a launch per tile shape, in us:
//   fixed + rounds * (K/64 * full + epi) + K/64 * (lone + (full - lone) * r) + epi * (1 + r) / 2
// where a round fills `slots` workgroups on each of the 256 CUs of a whole device
// (another count changes the speed of the choice, not a result), r is the
// filled part of the last round (left out when 0), `lone` and `full` are the
// time per K slice of 64 of a tile alone on its CU and of a full chip, and epi
// grows by epi_res for residual updates.  The constants are a least-squares fit
// to 966 measured shapes (32 to 65,520 rows; N and K of projections at widths
// 128 to 5120 and of the heads; bf16 stores and residual updates), each launch
// on another copy of the weights out of 900 MB: in a model a layer's weights
// come from HBM, which shifts the choice towards shapes with more loads in
// flight.  They were then adjusted for the choice rather than for the times:
// against the best tile of each of these shapes (none was held out) it costs 1.0%
// on average below 1,024 rows or so (at most 20%, at launches of 20 us) and 0.6%
// above, where 256 x 256 tiles for everything took 3.2 times and 12% longer on
// average.  A 128 x 256 tile is not among them, though at width 5120 it measured 4
// to 8% faster than the tile chosen (1024 x 5120 x 13824 190 against 205 us, 3120 x
// 5120 x 5120 152 against 160).  The row counts between 128 and 256 are for the
// last round: 12,480 x 1536 x 8960 takes 384 us with 256 rows (294 workgroups on
// 256 CUs), 315 with 192 and 297 with 160 (468, two nearly full rounds), 12,480 x
// 4608 x 1536 154 us with 256 and 144 with 224.
struct TileCost { int bm, bn, slots; double lone, full, fixed, epi, epi_res; };
static constexpr TileCost TILE_COST[N_TILES] = {
    {256, 256, 1, 1.022, 1.378, 3.20, 6.88, 16.20},
    {224, 256, 1, 0.820, 1.222, 1.71, 6.29, 14.71},
    {192, 256, 1, 0.785, 1.107, 3.09, 5.48, 11.52},
    {160, 256, 1, 0.754, 0.977, 1.74, 3.78, 9.75},
    {128, 128, 2, 0.472, 0.930, 2.00, 2.62, 5.00},
    {64, 64, 3, 0.246, 0.646, 2.07, 1.14, 0.88},
    {128, 128, 1, 0.469, 0.457, 1.29, 4.23, 2.50},
    {64, 128, 1, 0.355, 0.368, 1.56, 2.16, 0.92},
    {64, 64, 1, 0.198, 0.218, 1.79, 1.51, 0.41},
    {32, 64, 2, 0.164, 0.276, 1.86, 1.05, 0.25},
    {32, 32, 2, 0.159, 0.245, 1.76, 0.76, 0.00},
};

// The loop is unrolled so that every division is by a constant (0.07 us a launch
// instead of 0.12).
static Bf16Tile choose_tile(long M, long N, long K, long batch, bool residual) {
  const double nk = (double)(K / 64);
  auto cost = [&](int i) {
    const TileCost& c = TILE_COST[i];
    const long tiles = (M + c.bm - 1) / c.bm * ((N + c.bn - 1) / c.bn) * batch, round = 256L * c.slots;
    const double epi = c.epi + (residual ? c.epi_res : 0.0), r = (double)(tiles % round) / (double)round;
    double t = c.fixed + (double)(tiles / round) * (nk * c.full + epi);
    if (r > 0) t += nk * (c.lone + (c.full - c.lone) * r) + epi * 0.5 * (1.0 + r);
    return t;
  };
  int best = 0;
  double best_t = cost(0);
#pragma clang loop unroll(full)
  for (int i = 1; i < N_TILES; ++i) {
    const double t = cost(i);
    if (t < best_t) { best = i; best_t = t; }
  }
  return (Bf16Tile)best;
}

}  // namespace cs
