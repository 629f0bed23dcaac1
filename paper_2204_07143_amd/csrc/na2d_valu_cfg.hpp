// LDS footprints and tile heights of the plain-ALU 2D kernels (fp32), and which problems they serve.
#pragma once

#include "na2d_common.hpp"
#include "na2d_kernels.hpp"
#include "na2d_tile.hpp"

namespace na2d {

constexpr int kLdsLimit = 160 * 1024;

template <int K, int TY, int D>
struct QkCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int NB = 2 * K - 1;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<float, D>::kKeyStride;
    static constexpr int kBiasBytes = ((NB * NB * 4) + 15) & ~15;
    static constexpr int kRowRegion = mirror_bytes(kTileX * KK * (int)sizeof(float));
    static constexpr int kLdsBytes = kHaloBytes + kBiasBytes + TY * kRowRegion;
};

template <int K, int TY, int D>
struct AvCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<float, D>::kKeyStride;
    static constexpr int kRowRegion = mirror_bytes(kTileX * KK * (int)sizeof(float));
    static constexpr int kLdsBytes = kHaloBytes + TY * kRowRegion;
};

template <int K, int TY, int D>
struct InvCfg {
    // Query rectangle of a tile: at most tile + (K-1) + (K-1)/2 on an axis unless the tile
    // touches both borders of a short axis; the rare remainder is read from global memory.
    static constexpr int RECT_H = TY + K - 1 + K / 2, RECT_W = kTileX + K - 1 + K / 2;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kLdsBytes = RECT_H * RECT_W * VecTraits<float, D>::kKeyStride;
};

template <int K, int TY, int D>
struct FusedCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int NB = 2 * K - 1;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<float, D>::kKeyStride;
    static constexpr int kBiasBytes = ((NB * NB * 4) + 15) & ~15;
    static constexpr int kLdsBytes = 2 * kHaloBytes + kBiasBytes;
};

// Tile height: the one that keeps the most waves resident on a compute unit (workgroups that fit the LDS x waves
// per workgroup, at most 32 waves), the taller tile on a tie (its halo is shared by more queries; measured faster).
template <template <int, int, int> class Cfg, int K, int D>
constexpr int tile_rows() {
    int best = 4, best_waves = 0;
    const int lds[3] = {Cfg<K, 4, D>::kLdsBytes, Cfg<K, 8, D>::kLdsBytes, Cfg<K, 16, D>::kLdsBytes};
    for (int i = 0; i < 3; ++i) {
        const int ty = 4 << i, waves_per_wg = ty * kTileX / kWave;
        int wgs = lds[i] > 0 ? kLdsLimit / lds[i] : 0;
        int waves = wgs * waves_per_wg;
        waves = waves > 32 ? 32 : waves;
        if (waves >= best_waves && waves > 0) {
            best = ty;
            best_waves = waves;
        }
    }
    return best;
}
template <template <int, int, int> class Cfg, int K, int D>
constexpr bool tile_fits() {
    return Cfg<K, tile_rows<Cfg, K, D>(), D>::kLdsBytes <= kLdsLimit;
}

// Which problems run these kernels: fp32 (16 bit is the matrix cores' throughout), a window that is not too wide for the
// head dim, and from a number of strips (na2d_strip.hip) on: the strips' time grows with their number, whatever part of
// their 16 positions lies in the map, while below 1300 or so the chip is idle and a tile's one thread per query waits for
// LDS.  A row of one strip (W <= 16) takes its window rows in one block of keys instead of two, so the strips that load or
// store weights win sooner there.  Measured over 54k fp32 problems (D = 16, 32, 64, k = 3 .. 13, 16 maps from 7 x 7 to
// 200 x 334, 500 to 500k queries); time of the strips over that of the tiles, medians on maps of more than 60k queries:
//   logits        D = 16, k = 3 .. 9 wide maps 2.0, 1.9, 1.5, 1.0 (k = 11: 0.5); W <= 16: 1.6, 1.4, 1.1, 0.8;
//                 D = 32, k = 3 .. 7 1.8, 1.6, 1.1 (k = 9: 0.6); 1.3, 1.1, 0.8;  D = 64 1.0, 1.0; 0.7, 0.7
//   weighted sum  D = 16, k = 3 .. 9 1.6, 1.8, 1.6, 1.3 (k = 11: 0.7); 1.4, 1.2, 0.9, 0.7;
//                 D = 32, k = 3 .. 7 1.3, 1.4, 1.0 (0.8 .. 1.2); 1.0, 0.9, 0.6;  D = 64 0.8
//   inverse       D = 16, k = 3 .. 7 1.7, 1.1, 0.7; 1.3, 0.8, 0.5;  D = 32 1.3, 0.9, 0.4; 1.0, 0.6
//   fused         against the patches of na2d_patch_fwd.hip (100k queries on 14 x 14, 33 x 70 and 56 x 56 maps; their time over that of the
//                 tiles): D = 16, k = 3 .. 7 1.3 .. 1.6, 1.0 .. 1.5, 0.97 .. 1.36 (k = 9: 0.58 .. 0.71);  D = 32 0.82 .. 0.97, 0.54 .. 0.73
// and they cross where strips are few (same maps): fused 1300 to 1800 strips (then against strips), logits 1300 to 2000 (W <= 16: 2500), weighted
// sum 1500 to 2500 (3000 to 4000), inverse 3000; at the widest windows with tiles both ways win in turns up to 6000.  With this
// rule a problem takes 0.6 % longer on average than with the faster of the two, and 0.2 % of them run more than a tenth slower
// than in tiles; with one line at 32768 queries for all of them it was 2.2 % and 1.2 % (fused D = 16, k = 5, 458 7 x 7
// maps 18.8 us where the tiles take 9.3).
enum class ValuOp { logits, weighted_sum, inverse, fused };
constexpr int kNoTiles = 0x7fffffff;
// strips from which on the tiles are taken
constexpr int valu_least_strips(ValuOp op, int D, int K, bool one_strip_rows) {
    const int quick = K <= 5 && D <= 32 ? 1280 : 1536;
    switch (op) {
        case ValuOp::logits:
            if (one_strip_rows) return K <= (D == 16 ? 7 : D == 32 ? 5 : 0) ? 2560 : kNoTiles;
            return K <= (D == 16 ? 9 : D == 32 ? 7 : D == 64 ? 5 : 0) ? quick : kNoTiles;
        case ValuOp::weighted_sum:
            if (one_strip_rows) return K <= (D == 16 ? 5 : D == 32 ? 3 : 0) ? 3072 : kNoTiles;
            return K <= (D == 16 ? 9 : D == 32 ? 5 : 0) ? 1536 : D == 32 && K == 7 ? 2560 : kNoTiles;
        case ValuOp::inverse:
            if (one_strip_rows) return D == 16 && K == 3 ? 4096 : kNoTiles;
            return K == 3 && D <= 32 ? 3072 : D == 16 && K == 5 ? 6144 : kNoTiles;
        default: return K <= (D == 16 ? 7 : 0) ? quick : kNoTiles;
    }
}
constexpr bool valu_has_tile(ValuOp op, int D, int K) { return valu_least_strips(op, D, K, false) != kNoTiles; }
inline bool valu_preferred(const Problem &p, ValuOp op) {
    const int least = valu_least_strips(op, p.D, p.K, p.W <= kStrip);
    return p.dtype == NA2D_F32 && least != kNoTiles && p.strips() >= least;
}

}  // namespace na2d
