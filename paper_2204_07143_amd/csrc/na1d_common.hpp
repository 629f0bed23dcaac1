// Device code that the 1D kernels share.
#pragma once

#include "na2d_common.hpp"
#include "na2d_mfma.hpp"

namespace na1d {

using namespace na2d;

// The bias gradient's fixed point: 42 fraction bits
__device__ __forceinline__ long long to_fixed42(float x) {
    float y = x * 1024.f;
    if (!(__builtin_fabsf(y) < 2147483520.f)) y = 0.f;   // non-finite or out of range: counts as 0
    const float fl = __builtin_floorf(y);
    return (long long)(((unsigned long long)(uint32_t)(int)fl << 32) | (uint32_t)((y - fl) * 4294967296.f));
}
__device__ __forceinline__ long long to_fixed42(double x) {   // (in range)
    const double y = x * 1024., fl = __builtin_floor(y);
    return (long long)(((unsigned long long)(uint32_t)(int)fl << 32) | (uint32_t)((y - fl) * 4294967296.));
}

// The last sum of the bias gradient: the tables that the workgroups of a (batch, tile) left, added per head and cell (integers: any order).  A
// workgroup of kFinalThreads per cell, of a kernel of its own or at the end of the grid of the kernel that follows the one that leaves the tables.
constexpr int kFinalThreads = 256;
struct RpbTables {
    const long long *partial;
    BiasOut d_rpb;
    int B, heads, tiles, NB;
};
hipError_t launch_rpb_final(const RpbTables &p, hipStream_t s);
__device__ __forceinline__ void rpb_final_cell(const RpbTables &p, int block, int lds) {   // lds: 8 bytes per wave
    const int h = block / p.NB, u = block - h * p.NB, total = p.B * p.tiles;
    long long sum = 0;
    for (int n0 = threadIdx.x; n0 < total; n0 += 4 * kFinalThreads) {
        long long v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + j * kFinalThreads;
            v[j] = n < total ? p.partial[(((size_t)(n / p.tiles) * p.heads + h) * p.tiles + n % p.tiles) * p.NB + u] : 0ll;
        }
        sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int sh = 1; sh < kWave; sh <<= 1) sum += __shfl_xor(sum, sh, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) *lds_ptr<long long>(lds + threadIdx.x / kWave * 8) = sum;
    workgroup_sync();
    if (threadIdx.x == 0) {
        long long tot = 0;
        for (int w = 0; w < kFinalThreads / kWave; ++w) tot += *lds_ptr<long long>(lds + w * 8);
        p.d_rpb.store((size_t)h * p.NB + u, (float)((double)tot * (1.0 / 4398046511104.0)));   // 2^-42
    }
}

// Where a running maximum starts: not -inf, whose difference to a first logit of -inf (a masked bias cell) would be NaN
constexpr float kLowest = -3.402823466e38f;

// ---- matrix-core kernels (16 bit) ------------------------------------------------------------
constexpr int kGroup = 16, kBytes = 64;   // positions of a group, bytes of a head vector
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
// Weights enter products as two 16-bit halves; in fp16 they are scaled by 2^15 first, for the second not to fall below the type's
// smallest numbers.
template <typename T> constexpr float kShift = Traits<T>::kDtype == NA2D_F16 ? 15.f : 0.f;

template <typename T> __device__ __forceinline__ uint32_t pack2(float a, float b) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef T tx2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, tx2_t));
}
// x rounded to T (two per word) and what the rounding left
template <typename T> __device__ __forceinline__ void split2(float a, float b, uint32_t &hi, uint32_t &lo) {
    typedef T tx2_t __attribute__((ext_vector_type(2)));
    hi = pack2<T>(a, b);
    const tx2_t h = __builtin_bit_cast(tx2_t, hi);
    lo = pack2<T>(a - (float)h[0], b - (float)h[1]);
}
template <typename T> struct Split4 {   // a lane's four weights against a block
    uint32_t hi[2], lo[2];
    __device__ __forceinline__ void set(const float (&w)[4]) {
        split2<T>(w[0], w[1], hi[0], lo[0]);
        split2<T>(w[2], w[3], hi[1], lo[1]);
    }
};
// Against 64 bits the forward's and the backward's results with halves have the 2-norm error of those with whole fp32 weights to 1e-5 of it (1.66e-3 in
// bf16, 2.07e-4 in fp16: the result's own rounding; k = 3 .. 63, 16 cases of zero-mean inputs; dq in fp16 with offsets of 3 in k and v and 1 in q 2 to 3 % more).
// acc += (vectors of NBLK blocks, transposed) x weights; addr: the lane's part of block 0 (see vector_addr).  All products have the full depth:
// with the half-depth instruction for an odd last block, behind full-depth ones in the same accumulators, one build left two of a lane's
// eight results wrong.
template <typename T, int NBLK> __device__ __forceinline__ void weighted_sum(int addr, const Split4<T> (&w)[NBLK], f32x4 (&acc)[2]) {
#pragma unroll
    for (int c = 0; c < NBLK; c += 2)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const u32x2 v0 = lds_read_tr16(addr + c * kGroup * kBytes + hf * 8);
            const bool two = c + 1 < NBLK;   // (an odd last block: the other half of the depth is zeros)
            const int d = two ? c + 1 : c;
            const u32x2 v1 = two ? lds_read_tr16(addr + d * kGroup * kBytes + hf * 8) : u32x2{0u, 0u};
            const u32x4 a{v0.x, v0.y, v1.x, v1.y};
            acc[hf] = mfma_16x16x32<T>(a, u32x4{w[c].lo[0], w[c].lo[1], two ? w[d].lo[0] : 0u, two ? w[d].lo[1] : 0u}, acc[hf]);
            acc[hf] = mfma_16x16x32<T>(a, u32x4{w[c].hi[0], w[c].hi[1], two ? w[d].hi[0] : 0u, two ? w[d].hi[1] : 0u}, acc[hf]);
        }
}
// where lane (j, g) reads position 0 of an image as operand rows and for the transposed sums (which leave it channels 8 g .. 8 g + 7)
__device__ __forceinline__ int row_addr(int img, int pos, int j, int g) { return img + (pos + j) * kBytes + g * 16; }
__device__ __forceinline__ int vector_addr(int img, int pos, int j, int g) { return img + (pos + 4 * g + (j >> 2)) * kBytes + (j & 3) * 16; }
template <typename T> __device__ __forceinline__ void store_vector(char *at, const float (&x)[8]) {
    store16_stream(at, u32x4{pack2<T>(x[0], x[1]), pack2<T>(x[2], x[3]), pack2<T>(x[4], x[5]), pack2<T>(x[6], x[7])});
}
// `rows` (a multiple of 16) head vectors of two tensors from a and b on into two images by direct loads, 16 to a piece, the pieces to the waves
// in turn; past `last` the vector there again (it only meets zero weights)
template <int WAVES>
__device__ __forceinline__ void stage_pair(const char *a, const char *b, int last, int rows, int img_a, int img_b, int wave, int lane) {
    for (int p = wave; p < rows / kGroup; p += WAVES) {
        const int row = p * kGroup + (lane >> 2), at = row < last ? row : last;
        const unsigned off = (unsigned)(at * kBytes + (lane & 3) * 16);
        global_to_lds_16(a, off, img_a + p * kGroup * kBytes);
        global_to_lds_16(b, off, img_b + p * kGroup * kBytes);
    }
}
// x of the lane 16 (or 32) further, in one instruction that swaps halves instead of two trips through the LDS unit; the four lanes of a
// column are active together wherever this is called
template <int D> __device__ __forceinline__ void both_halves(float x, float &a, float &b) {
    typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
    const unsigned u = __float_as_uint(x);
    const u32x2_t r = D == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    a = __uint_as_float(r.x);
    b = __uint_as_float(r.y);
}
__device__ __forceinline__ float group_max(float x) {   // over the four lanes of a column
    float a, b;
    both_halves<16>(x, a, b);
    both_halves<32>(fmaxf(a, b), a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float group_sum(float x) {
    float a, b;
    both_halves<16>(x, a, b);
    both_halves<32>(a + b, a, b);
    return a + b;
}
template <typename T> __device__ __forceinline__ void load8_lds(VecN<T, 8> &v, int addr) {
    const u32x4 t = *lds_ptr<u32x4>(addr);
    v.w[0] = t.x, v.w[1] = t.y, v.w[2] = t.z, v.w[3] = t.w;
}
// Positions that the four lanes of a column look at together where a result is worked out once more: their reads and sums do not wait for each other.
constexpr int kOnceMore = 2;
// the columns (bit j) of which some lane is marked
__device__ __forceinline__ unsigned marked_columns(bool mark) {
    const unsigned long long m = __ballot(mark);
    return (unsigned)((m | (m >> 16) | (m >> 32) | (m >> 48)) & 0xffffu);
}

}  // namespace na1d
