// LDS footprints and tile heights of the plain-ALU 2D kernels, and which problems they serve.
#pragma once

#include "na2d_common.hpp"
#include "na2d_kernels.hpp"
#include "na2d_tile.hpp"

namespace na2d {

constexpr int kLdsLimit = 160 * 1024;

template <typename T, int K, int TY, int D = kHeadDim>
struct QkCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int NB = 2 * K - 1;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<T, D>::kKeyStride;
    static constexpr int kBiasBytes = ((NB * NB * 4) + 15) & ~15;
    static constexpr int kRowRegion = mirror_bytes(kTileX * KK * (int)sizeof(T));
    static constexpr int kLdsBytes = kHaloBytes + kBiasBytes + TY * kRowRegion;
};

template <typename T, int K, int TY, int D = kHeadDim>
struct AvCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<T, D>::kKeyStride;
    static constexpr int kRowRegion = mirror_bytes(kTileX * KK * (int)sizeof(T));
    static constexpr int kLdsBytes = kHaloBytes + TY * kRowRegion;
};

template <typename T, int K, int TY, int D = kHeadDim>
struct InvCfg {
    // Query rectangle of a tile: at most tile + (K-1) + (K-1)/2 on an axis unless the tile
    // touches both borders of a short axis; the rare remainder is read from global memory.
    static constexpr int RECT_H = TY + K - 1 + K / 2, RECT_W = kTileX + K - 1 + K / 2;
    static constexpr int KK = K * K;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kLdsBytes = RECT_H * RECT_W * VecTraits<T, D>::kKeyStride;
};

template <typename T, int K, int TY, int D = kHeadDim>
struct FusedCfg {
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    static constexpr int NB = 2 * K - 1;
    static constexpr int kThreads = kTileX * TY;
    static constexpr int kHaloBytes = HALO_H * HALO_W * VecTraits<T, D>::kKeyStride;
    static constexpr int kBiasBytes = ((NB * NB * 4) + 15) & ~15;
    static constexpr int kLdsBytes = 2 * kHaloBytes + kBiasBytes;
};

// Tile height: the one that keeps the most waves resident on a compute unit (workgroups that fit the LDS x waves
// per workgroup, at most 32 waves), the taller tile on a tie (its halo is shared by more queries; measured faster).
template <template <typename, int, int, int> class Cfg, typename T, int K, int D>
constexpr int tile_rows() {
    int best = 4, best_waves = 0;
    const int lds[3] = {Cfg<T, K, 4, D>::kLdsBytes, Cfg<T, K, 8, D>::kLdsBytes, Cfg<T, K, 16, D>::kLdsBytes};
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
template <template <typename, int, int, int> class Cfg, typename T, int K, int D>
constexpr bool tile_fits() {
    return Cfg<T, K, tile_rows<Cfg, T, K, D>(), D>::kLdsBytes <= kLdsLimit;
}

// Which problems run these kernels: fp32 (16 bit is the matrix cores' throughout), windows up to the side below, and
// enough queries that their large tiles fill the chip.  Measured on 56 x 56 maps, two heads, against the strip kernels
// (na2d_strip.hip), us, tile / strip: from 50k queries on the tiles win up to these sides (logits D = 32, k = 7:
// 18 / 27 at 50k and 91 / 123 at 300k queries; weighted sum 17 / 22 and 86 / 109; inverse D = 16, k = 5: 43 / 51 at
// 300k; fused D = 32, k = 7: 33 / 37 at 50k) and lose beyond them (k = 9: logits 219 / 161, weighted sum 200 / 138,
// inverse 341 / 115, fused 508 / 215 at 300k; D = 64, k = 9: 348 / 240, 463 / 196, 755 / 175, 1513 / 398; D = 128, k = 3:
// 220 / 148, 256 / 150, 275 / 147, 1010 / 336); at 25k and fewer the strips are as fast or faster at every side
// (inverse D = 32, k = 7 at 6k: 37 / 10).
enum class ValuOp { logits, weighted_sum, inverse, fused };
constexpr int valu_most_k(ValuOp op, int D) {
    switch (op) {
        case ValuOp::logits: return D == 16 ? 9 : D == 32 ? 7 : D == 64 ? 5 : 0;
        case ValuOp::weighted_sum: return D == 16 ? 9 : D == 32 ? 7 : 0;
        case ValuOp::inverse: return D == 16 ? 5 : D == 32 ? 3 : 0;
        default: return D == 16 ? 11 : D == 32 ? 7 : 0;
    }
}
constexpr size_t kValuQueries = 32768;
inline bool valu_preferred(const Problem &p, ValuOp op) {
    return p.dtype == NA2D_F32 && p.K <= valu_most_k(op, p.D) && p.queries() >= kValuQueries;
}

}  // namespace na2d
