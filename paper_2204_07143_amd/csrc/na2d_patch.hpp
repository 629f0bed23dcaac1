// Building blocks of the patch kernels (any window side, head dim and storage type): 4 x 4 patches of positions of one
// operand, kept in registers, against 4 x 4 blocks of positions of the other, streamed through LDS four map rows at a
// time (arXiv 2204.07143, Eq. 2-4: one small dense product per pair, masked by the window).
//
// Lane (column n = lane % 16, group g = lane / 16) of a wave holds position n of its patch (row n / 4, column n % 4) and
// receives the products with row g of a block, columns 0 .. 3.  In that layout the four products enter the matrix cores
// again as the weights of a sum over the block's positions.
#pragma once

#include "na2d_common.hpp"
#include "na2d_mfma.hpp"
#include "na2d_tile.hpp"

namespace na2d {

__device__ __forceinline__ f32x4 mfma_16x16x4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32v2 __attribute__((ext_vector_type(2)));

template <typename T> __device__ __forceinline__ uint32_t pack_pair(float a, float b) {
    typedef T tx2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, tx2_t));
}

// A head vector spread over the four lanes of a column, as an operand whose contraction runs over channels: chunks of 16
// bytes, chunk 4 i + g in lane group g (both operands alike, so the order of the channels is free).  16 channels in 16
// bit: eight bytes a lane and the half-depth instruction.
template <typename T, int D> struct ChanVec {
    static constexpr bool HALF = sizeof(T) == 2 && D == 16;
    static constexpr int kLaneBytes = HALF ? 8 : 16;                 // byte offset between lane groups
    static constexpr int N = HALF ? 1 : D * (int)sizeof(T) / 64;     // 16-byte chunks per lane
    u32x4 c[N];
    __device__ __forceinline__ void load(const char *lane_vec) {     // (the lane's first chunk)
        if constexpr (HALF) {
            const u32v2 t = *reinterpret_cast<const u32v2 *>(lane_vec);
            c[0] = u32x4{t.x, t.y, 0u, 0u};
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) c[i] = *reinterpret_cast<const u32x4 *>(lane_vec + i * 64);
        }
    }
    __device__ __forceinline__ void load_lds(int addr) {
        if constexpr (HALF) {
            const u32v2 t = *lds_ptr<u32v2>(addr);
            c[0] = u32x4{t.x, t.y, 0u, 0u};
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) c[i] = *lds_ptr<u32x4>(addr + i * 64);
        }
    }
};
// A value loaded from memory that is used behind direct-to-LDS loads: the compiler's wait for it goes here.  (It does not know
// those loads; a wait of its own further down would be for them too.)
template <typename T, int D> __device__ __forceinline__ void settle(ChanVec<T, D> &v) {
#pragma unroll
    for (int i = 0; i < ChanVec<T, D>::N; ++i) asm volatile("" : "+v"(v.c[i]));
}
// rows: the block's positions (a), columns: the patch's (b); from: what the products are added to
template <typename T, int D> __device__ __forceinline__ f32x4 chan_dot(const ChanVec<T, D> &a, const ChanVec<T, D> &b, f32x4 from = f32x4{0.f, 0.f, 0.f, 0.f}) {
    f32x4 acc = from;
    if constexpr (ChanVec<T, D>::HALF) {
        acc = mfma_16x16x16<T>(a.c[0].x, a.c[0].y, b.c[0].x, b.c[0].y, acc);
    } else if constexpr (sizeof(T) == 4) {
        // two chains of additions, half as long: closer to the exact product, and the matrix cores need not wait for one of them
        f32x4 odd{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < ChanVec<T, D>::N; ++i) {
            const f32x4 x = __builtin_bit_cast(f32x4, a.c[i]), y = __builtin_bit_cast(f32x4, b.c[i]);
            acc = mfma_16x16x4(x[0], y[0], acc);
            odd = mfma_16x16x4(x[1], y[1], odd);
            acc = mfma_16x16x4(x[2], y[2], acc);
            odd = mfma_16x16x4(x[3], y[3], odd);
        }
        acc += odd;
    } else {
#pragma unroll
        for (int i = 0; i < ChanVec<T, D>::N; ++i) acc = mfma_16x16x32<T>(a.c[i], b.c[i], acc);
    }
    return acc;
}

// The positions of a block as an operand whose contraction runs over positions (channels are its rows), and the sums
// built with it.  The channels are dealt over the rows so that a lane ends with eight consecutive channels
// 32 p + 8 g .. + 7 of its position per pair of accumulators (D = 16: four, 4 g .. + 3).
template <typename T, int D> struct PosOp {
    static constexpr int NA = D / 16;   // accumulators
    static constexpr int POSB = D * (int)sizeof(T);
    u32v2 c[sizeof(T) == 2 ? NA : 2 * NA];
    // this lane's address of block column 0 inside an image of `rw` positions per row
    __device__ static __forceinline__ int lane_offset(int lane, int rw) {
        const int j = lane & 15, g = lane >> 4;
        if constexpr (sizeof(T) == 2) return (g * rw + (j >> 2)) * POSB + (j & 3) * (D == 16 ? 8 : 16);
        return g * rw * POSB + j * (D == 16 ? 4 : 8);
    }
    __device__ __forceinline__ void load_lds(int addr) {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const u32x2 t = lds_read_tr16(addr + (i >> 1) * 64 + (i & 1) * 8);
                c[i] = u32v2{t.x, t.y};
            }
        } else if constexpr (D == 16) {
            c[0] = u32v2{*lds_ptr<uint32_t>(addr), *lds_ptr<uint32_t>(addr + POSB)};
            c[1] = u32v2{*lds_ptr<uint32_t>(addr + 2 * POSB), *lds_ptr<uint32_t>(addr + 3 * POSB)};
        } else {
#pragma unroll
            for (int p = 0; p < NA / 2; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) c[4 * p + e] = *lds_ptr<u32v2>(addr + e * POSB + p * 128);
        }
    }
};
template <typename T> struct Weights4 {   // the lane's four weights, in storage type (fp32: as they are)
    float f[sizeof(T) == 4 ? 4 : 1];
    uint32_t p0, p1;
    Weights4() = default;
    __device__ __forceinline__ explicit Weights4(const float (&w)[4]) {
        if constexpr (sizeof(T) == 2) {
            p0 = pack_pair<T>(w[0], w[1]);
            p1 = pack_pair<T>(w[2], w[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = w[e];
        }
    }
};
template <typename T, int D> struct PosSum {
    using Op = PosOp<T, D>;
    f32x4 acc[Op::NA];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < Op::NA; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add(const Op &o, const Weights4<T> &w) {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < Op::NA; ++i) acc[i] = mfma_16x16x16<T>(o.c[i].x, o.c[i].y, w.p0, w.p1, acc[i]);
        } else if constexpr (D == 16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0] = mfma_16x16x4(__uint_as_float((e & 1) ? o.c[e >> 1].y : o.c[e >> 1].x), w.f[e], acc[0]);
        } else {
#pragma unroll
            for (int p = 0; p < Op::NA / 2; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[2 * p] = mfma_16x16x4(__uint_as_float(o.c[4 * p + e].x), w.f[e], acc[2 * p]);
                    acc[2 * p + 1] = mfma_16x16x4(__uint_as_float(o.c[4 * p + e].y), w.f[e], acc[2 * p + 1]);
                }
        }
    }
    __device__ __forceinline__ void take(PosSum &part) {   // adds another's sums and clears them
        part.settle();
#pragma unroll
        for (int i = 0; i < Op::NA; ++i) {
            acc[i] += part.acc[i];
            part.acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // two blocks: in 16 bit one full-depth product for both
    __device__ __forceinline__ void add2(const Op &o0, const Weights4<T> &w0, const Op &o1, const Weights4<T> &w1) {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < Op::NA; ++i)
                acc[i] = mfma_16x16x32<T>(u32x4{o0.c[i].x, o0.c[i].y, o1.c[i].x, o1.c[i].y}, u32x4{w0.p0, w0.p1, w1.p0, w1.p1}, acc[i]);
        } else {
            add(o0, w0);
            add(o1, w1);
        }
    }
    // one block behind add2()'s: the full depth again, zeros in its other half (16 bit: accumulators meet one instruction only, see the 1D
    // kernels' weighted_sum)
    __device__ __forceinline__ void add_last(const Op &o, const Weights4<T> &w) {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < Op::NA; ++i) acc[i] = mfma_16x16x32<T>(u32x4{o.c[i].x, o.c[i].y, 0u, 0u}, u32x4{w.p0, w.p1, 0u, 0u}, acc[i]);
        } else {
            add(o, w);
        }
    }
    __device__ __forceinline__ void settle() { settle_products<Op::NA>(acc); }
    // NaN if any sum of the lane is not finite, 0 otherwise
    __device__ __forceinline__ float not_finite() const {
        float c = 0.f;
#pragma unroll
        for (int i = 0; i < Op::NA; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) c = __builtin_fmaf(acc[i][r], 0.f, c);
        return c;
    }
    // the lane's part of the head vector at base + off
    __device__ __forceinline__ void store(char *base, unsigned off, int g, float f) const {
        if constexpr (D == 16) {
            if constexpr (sizeof(T) == 2) {
                *reinterpret_cast<u32v2 *>(base + (off + g * 8)) = u32v2{pack_pair<T>(acc[0][0] * f, acc[0][1] * f), pack_pair<T>(acc[0][2] * f, acc[0][3] * f)};
            } else {
                store16_stream(base + (off + g * 16), __builtin_bit_cast(u32x4, acc[0] * f));
            }
        } else {
            off += g * (sizeof(T) == 2 ? 16 : 32);
#pragma unroll
            for (int p = 0; p < Op::NA / 2; ++p) {
                const f32x4 a = acc[2 * p] * f, b = acc[2 * p + 1] * f;
                if constexpr (sizeof(T) == 2) {
                    store16_stream(base + (off + p * 64), u32x4{pack_pair<T>(a[0], a[1]), pack_pair<T>(a[2], a[3]),
                                                               pack_pair<T>(b[0], b[1]), pack_pair<T>(b[2], b[3])});
                } else {
                    store16_stream(base + (off + p * 128), __builtin_bit_cast(u32x4, f32x4{a[0], b[0], a[1], b[1]}));
                    store16_stream(base + (off + p * 128 + 16), __builtin_bit_cast(u32x4, f32x4{a[2], b[2], a[3], b[3]}));
                }
            }
        }
    }
};

// `rows` (4, 8, 16 or 32) consecutive map rows of one plane of two tensors, `rw` positions each from column x0 on, into two LDS images
// (the second img_bytes behind the first) by direct loads.  Positions outside the map are replaced by the nearest one inside it (they
// only meet zero weights).  A row's 1 KB pieces go to the waves of a workgroup in turn (two waves to a row while there are four;
// rw is a whole number of pieces).
constexpr int kPatchWaves = 8, kPatchThreads = kPatchWaves * kWave;
template <int POSB> constexpr int kRowUnit = POSB >= 1024 ? 1 : 1024 / POSB;   // positions per piece
template <int POSB>
__device__ __forceinline__ void issue_rows(const char *plane_a, const char *plane_b, int H, int W, int y0, int x0, int rw, int img, int img_bytes, int wave, int lane,
                                           int rows = 4) {
    constexpr int CPP = POSB / 16;
    // (recomputed at every call: as loop invariants the addresses below would spill scalar registers)
    asm volatile("" : "+s"(rw), "+s"(W), "+s"(wave));
    const int per_row = rows == 4 ? 2 : 1, first = rows == 4 ? wave >> 2 : 0;
    for (int row = rows == 4 ? wave & 3 : wave; row < rows; row += kPatchWaves) {
        const unsigned line = (unsigned)((y0 + row < H - 1 ? y0 + row : H - 1) * W);   // (a plane is smaller than 2^31 bytes)
        const char *a = plane_a + (size_t)line * POSB, *b = plane_b + (size_t)line * POSB;
        int dst = img + (row * rw) * POSB + first * 1024;
        const int end = img + (row + 1) * rw * POSB;
        int x = x0 + first * kRowUnit<POSB> + lane / CPP;
        for (; dst < end; dst += per_row * 1024, x += per_row * kRowUnit<POSB>) {
            const unsigned off = (unsigned)((x < W - 1 ? x : W - 1) * POSB + (lane % CPP) * 16);
            global_to_lds_16(a, off, dst);
            global_to_lds_16(b, off, dst + img_bytes);
        }
    }
}

constexpr float kLog2e = 1.4426950408889634f, kLog2eLow = (float)(1.4426950408889634 - (double)kLog2e);
// scale2 s + bias with scale2 to twice its digits (an infinite s must not meet the infinity of the other sign)
__device__ __forceinline__ float exponent_fp32(float s, float scale2, float scale2_low, float bias) {
    return __builtin_fmaf(scale2, s, __builtin_fmaf(scale2_low, __builtin_amdgcn_fmed3f(s, -3e38f, 3e38f), bias));
}
// fp32 dot product of two head vectors in memory
template <typename T, int D> __device__ __forceinline__ float dot_memory(const T *a, const T *b) {
    float acc = 0.f;
#pragma unroll
    for (int d = 0; d < D; d += 8) {
        VecN<T, 8> x, y;
        load_vec32(x, a + d);
        load_vec32(y, b + d);
        acc += dot32(x, y);
    }
    return acc;
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}

// Slots of a rectangle in raster order, one after the other (past the last it stays there)
struct RasterWalk {
    int row = 0, col = 0;
    __device__ __forceinline__ void next(int rows, int cols) {
        const bool wrap = col == cols - 1, more = row < rows - 1;
        col = !wrap ? col + 1 : more ? 0 : col;
        row += wrap && more;
    }
};
// A result worked out once more takes the place of one that is not finite; the others, added up in another order, stay.
template <typename T> __device__ __forceinline__ void replace_not_finite(T *at, float x) {
    if (!(fabsf(to_f32(*at)) < INFINITY)) *at = from_f32<T>(x);
}
// Image buffers: two while two workgroups then share a compute unit, one where that is what lets two share it (or what fits at all); 0: too large
static inline int image_buffers(int fixed, int stage, int &lds_bytes) {
    constexpr int kCu = 160 * 1024;
    const int n = fixed + 2 * stage <= kCu / 2 || (fixed + stage > kCu / 2 && fixed + 2 * stage <= kCu) ? 2 : 1;
    lds_bytes = fixed + n * stage;
    return lds_bytes <= kCu ? n : 0;
}
// The bias table in LDS: rows of bias_pitch() fp32 entries, kBiasPad of padding (zeros) in front of entry 0 and as much
// behind the last; a patch's products reach that far beyond the table outside their windows.  The pitch is 8 mod 32 so that the
// rows a wave reads at once start in different banks.  One more row holds -inf: where a lane's row of a block is not in its
// window it reads its bias there, and its weights become 0 without a test.  Without a bias there is one row of zeros before it.
constexpr int kBiasPad = 6;
__host__ __device__ constexpr int bias_pitch(int K) { return (2 * K - 1 + 2 * kBiasPad - 8 + 31) / 32 * 32 + 8; }
__host__ __device__ constexpr int bias_rows(int K, bool with_bias) { return (with_bias ? 2 * K - 1 : 1) + 1; }
// the head's bias table times log2(e)
template <typename T>
__device__ __forceinline__ void stage_bias(const T *table, int K, FastDiv by_pitch, int bias0, int tid) {
    const int NB = 2 * K - 1, pitch = bias_pitch(K), rows = table ? NB : 1;
    for (int i = tid; i < (rows + 1) * pitch; i += kPatchThreads) {
        const int u = fdiv(i, by_pitch), v = i - u * pitch - kBiasPad;
        float x = u == rows ? -INFINITY : 0.f;
        if (table && u < rows && (unsigned)v < (unsigned)NB) x = to_f32(table[u * NB + v]) * 1.4426950408889634f;
        *lds_ptr<float>(bias0 + i * 4) = x;
    }
}
// LDS base of the launch's dynamic memory, as a value the compiler keeps in a register instead of adding it to every address
__device__ __forceinline__ int dynamic_lds(const char *lds) {
    int a = lds_addr(lds);
    asm volatile("" : "+s"(a));
    return a;
}

struct PatchShape {
    int H, W, K, heads, tiles_y, units, splits;
    int rw;                // positions per image row
    int lg_split;          // 2^lg_split waves share a patch, each with its rows of blocks (forward; backward, key side: 0 or 1)
    int lg_cols;           // a tile is 2^lg_cols patches wide and (8 >> lg_split) / 2^lg_cols patches high
    int nstage;            // LDS buffers (1: reloaded between steps)
    int copies;            // of the integer bias gradients
    int with_bias, with_dbias;
    GridDecode gd;
    FastDiv by_pitch;
    int two;               // backward in 16 bit: part 2 takes two patches to a wave (and what part 1 leaves for it)
};

// Host: positions per image row for tiles of `tw` columns on a map of `W`: what the widest tile's patches reach from the image's first
// column, in whole pieces.  `first` and `last`: the first and the last position of the streamed operand that a position of the kept one
// meets; a wave's patches are `step` columns wide.  Tiles clear of both borders are alike: of those one is enough.
template <typename First, typename Last> inline int image_row(int W, int K, int tw, int posb, First first, Last last, int step = 4) {
    int rw = 0;
    const int border = 2 * K + 2 * tw, skip_to = (W - border) / tw * tw;   // (at least a tile of the middle is looked at)
    for (int px = 0; px < W; px += step) {
        if (px >= border + tw && px < skip_to) px = skip_to;
        const int px3 = px + step - 1 < W - 1 ? px + step - 1 : W - 1, o = first(px);
        const int e = o - first(px / tw * tw) + ((last(px3) - o + 4) & ~3);
        rw = rw > e ? rw : e;
    }
    const int unit = 1024 / posb > 1 ? 1024 / posb : 1;
    return (rw + unit - 1) / unit * unit;
}

}  // namespace na2d
