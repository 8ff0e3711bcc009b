// The tile of the projection GEMM for an output size: plain C++, no HIP, for
// the launcher and for host tests.
#pragma once

#include <cstdint>

namespace hcms {

// The tiles, and what a round of workgroups and a stage of 128 bytes of K
// take on them, in us, measured (bf16; fp32 stages, as many bytes, take about
// as long): a stage with every CU busy, at the clock the power limit leaves,
// and with few of them busy, where the latency of the loads shows; and the
// start and the epilogue of a round.  Larger tiles move fewer bytes per MFMA,
// smaller ones keep more stages in flight and fill the CUs on smaller
// outputs: on 8192 x 8192 x 4096 the first takes 396 us, the others 440, 438,
// 495, 668 and 764; on 1560 x 5120 x 5120 99, 91, 86, 121, 123 and 140; on
// 1560 x 1920 x 5120 97, 82, 81, 41, 56 and 53; on 500 x 2000 x 4096 73, 58,
// 60, 28, 22 and 17.
struct TileCost {
    int bm, bn, per_cu;
    double full, alone, fixed;
};
inline constexpr TileCost kTiles[] = {
    {256, 256, 1, 1.50, 0.99, 5.0}, {192, 256, 1, 1.18, 0.82, 4.5}, {256, 192, 1, 1.18, 0.82, 4.5},
    {128, 128, 1, 0.49, 0.35, 2.0}, {64, 128, 1, 0.34, 0.26, 1.2},  {64, 64, 2, 0.37, 0.19, 1.2}};

// The tile with the shortest estimated time, from tile `first` on: whole
// rounds of workgroups, then a partial one whose stages lie between the two
// measured times.
inline int pick_tile(int64_t M, int64_t N, int64_t stages, int64_t n_cu, int first) {
    int best = first;
    double t_best = 0;
    for (int i = first; i < static_cast<int>(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const TileCost &c = kTiles[i];
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const int64_t slots = n_cu * c.per_cu, rem = tiles % slots;
        const double f = static_cast<double>(rem) / slots;
        double t = (tiles / slots) * (c.fixed + stages * c.full);
        if (rem > 0) t += c.fixed + stages * (c.alone + (c.full - c.alone) * f);
        if (i == first || t < t_best) {
            best = i;
            t_best = t;
        }
    }
    return best;
}

// The tile that launches take: kTiles[linear_tile(...)].  The rotation of fp32
// features does not fit beside the 256 x 256 tile's accumulators and staged
// values.
inline int linear_tile(int64_t M, int64_t N, int64_t K, int elem_bytes, bool qkv, int64_t n_cu) {
    return pick_tile(M, N, K * elem_bytes / 128, n_cu, qkv && elem_bytes == 4 ? 1 : 0);
}

}  // namespace hcms
