// Backward of neighbourhood attention without the k * k tensors, for any window side, head dim and storage type
// (arXiv 2204.07143: Eq. 2-4 differentiated): what na2d_fused_bwd.hip is for narrow windows of 16 and 32 channels in 16 bit,
// with the window side as a run-time argument and the rows of the streamed operand passing through LDS four at a time, so that
// neither the window nor the head dim is limited by a whole halo.
//
//   P[i, j] = exp(scale <q_i, k_j> + B(i, j) - lse_i)   dP[i, j] = <dout_i, v_j>   delta_i = sum_j P dP   dS = P (dP - delta)
//
// Part 1 keeps 4 x 4 query patches and streams keys and values once: delta and
//   dq_i = scale sum_j dS k_j = scale (sum_j P dP k_j - delta_i sum_j P k_j)
// so that delta need not be known before the sums (a second sweep would evaluate both products again).  In 16 bit P dP and P are
// rounded to the storage type, as the stored dp and the stored weights of the unfused steps are.  Where the dP of a window have much in
// common (values with an offset per channel, as a projection with a bias leaves them) the two sums would be large and nearly equal: dP and delta
// count from near_mean() of the query, which costs one product per patch and plane.
// Part 2 keeps 4 x 4 key patches and streams queries, upstream gradients, lse and delta: dv_j = sum_i P dout_i,
// dk_j = scale sum_i dS q_i, and the bias gradient: every dS is added to its cell of a table in LDS, as an integer (additions of
// integers commute: the result is bitwise reproducible).  Their scale follows a bound of the |dS|
// that the workgroup meets in a plane (part 1 leaves one per query patch, which its queries that are not finite have no part in); see BiasSums.
//
// A masked product is 0 * x: where x is not finite it would spoil positions whose window does not hold it, so results that are not
// finite are computed once more from their own window only.
// Measured (us, both parts and the bias gradient, in brackets the steps before: weights recomputed into memory and the unfused backward):
// 64 x 2 x 56 x 56 queries, fp16, 32 channels, k = 13 78 + 118 + 5 (455); fp32, k = 7 196 + 217 + 6 (700); fp16, 64 channels (one head), k = 7 48 + 65 + 9
// (165); 4 x 2 x 64 x 64, bf16, k = 21 18 + 40 + 4 (220).  By counters with one patch to a wave part 1 issues 60 vector
// instructions per 16 x 16 products, of which a block needs 40, and waits 43 % of its wave cycles: its four waves per SIMD do not cover the chain from LDS
// through two products, the exponential and two more.  Part 2 adds the integer additions in LDS.  In 16 bit large calls take two patches to a wave.  fp32 is
// nearer to its matrix cores: 32 instructions of 32 cycles per block, 94 us a part.
#include <limits.h>

#include "na2d_kernels.hpp"
#include "na2d_patch.hpp"

namespace na2d {

namespace {

// What part 1 leaves of a query for part 2: the base of its exponents and delta.  In 16 bit the base is log2(e) lse.  In fp32 it is 0
// (log2(e) lse rounded to a whole number where that is beyond +-32), and the inverse of the sum of the exponentials to that base
// follows (and a word of padding): P = exp2(t - base) / sum has neither the rounding of lse nor that of the difference in it.
// For the kernel with two patches to a wave (PatchShape::two): what its products start from, -lse / scale of all of a plane's queries, then
// -delta of all of them, so that exp2(scale2 (s + start) + bias) and dP need no further subtraction and four neighbours lie in a row.  The others read
// pairs: they are 2 to 4 % slower with the starts.
template <typename T> constexpr bool kNormalised = sizeof(T) == 4;
template <typename T> constexpr int kQueryWords = kNormalised<T> ? 4 : 2;

// waves per SIMD the kernels are built for: two workgroups per compute unit where 128 registers hold a wave
template <typename T, int D> constexpr int kPatchOcc = D * sizeof(T) <= 128 ? 4 : 2;

// blocks of a row whose loads are in flight together: two where the registers hold them
template <typename T, int D> constexpr int kAtOnceQ = (sizeof(T) == 2 && D <= 32) || kPatchOcc<T, D> == 2 ? 2 : 1;
template <typename T, int D> constexpr int kAtOnceKv = (sizeof(T) == 2 && D <= 32) || kPatchOcc<T, D> == 2 ? 2 : 1;

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int m = 1; m < kWave; m *= 2) x += __shfl_xor(x, m);
    return x;
}
template <int CTRL> __device__ __forceinline__ uint32_t dpp_max(uint32_t x) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
    return x > o ? x : o;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {   // (the exchanges inside the vector ALU, see column_sum)
    x = dpp_max<0xB1>(x);    // lane ^ 1
    x = dpp_max<0x4E>(x);    // lane ^ 2
    x = dpp_max<0x141>(x);   // the other half of eight lanes
    x = dpp_max<0x140>(x);   // the other half of sixteen
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = a[0] > a[1] ? a[0] : a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return b[0] > b[1] ? b[0] : b[1];
}
// |dS| = P |dP - delta| is at most this, given the largest P |dP| and P of the window; as bits (finite where delta is, infinity or NaN elsewhere)
__device__ __forceinline__ uint32_t ds_bound(float most_pdp, float most_p, float delta) {
    const float most = fabsf(__builtin_fmaf(most_p, fabsf(delta), most_pdp));
    return __float_as_uint(fabsf(delta) < INFINITY ? fminf(most, 3.4028234e38f) : most);
}
constexpr uint32_t kNotFinite = 0x7f800000u, kMark = 0x80000000u;
// Weight and upstream product of one (query, key) pair, from memory.
template <typename T, int D> struct PlanePtrs {
    const T *q, *k, *v, *dout, *rpb;   // of the plane; the head's bias table or null
};
template <typename T, int D>
__device__ __forceinline__ void pair_weight(const PlanePtrs<T, D> &m, const PatchShape &g, float scale, int iy, int ix, int y, int x,
                                            float base, float &p, float &dp) {
    const size_t i = ((size_t)iy * g.W + ix) * D, j = ((size_t)y * g.W + x) * D;
    float s = scale * dot_memory<T, D>(m.q + i, m.k + j);
    if (m.rpb) s += to_f32(m.rpb[(y - iy + g.K - 1) * (2 * g.K - 1) + x - ix + g.K - 1]);
    p = __builtin_amdgcn_exp2f(__builtin_fmaf(s, kLog2e, -base));
    dp = dot_memory<T, D>(m.dout + i, m.v + j);
}

// delta, dq and the bound of one query from its own window (a wave works on it: 64 window slots at a time, then a channel to
// a lane).  A delta that is NaN makes every dS NaN, so the sums need not be formed.
template <typename T, int D>
__device__ __forceinline__ float query_once_more(const PlanePtrs<T, D> &m, const PatchShape &g, float scale, int iy, int ix, float base, T *dq, uint32_t &bound, float &inv) {
    const int lane = threadIdx.x % kWave, K = g.K, KK = K * K, sy = win_start(iy, g.H, K), sx = win_start(ix, g.W, K);
    float delta = 0.f, z = 0.f;
    uint32_t most = 0, most_p = 0;
    for (int first = 0; first < KK; first += kWave) {
        const int slot = first + lane < KK ? first + lane : KK - 1, a = slot / K, c = slot - a * K;
        float p, dp;
        pair_weight(m, g, scale, iy, ix, sy + a, sx + c, base, p, dp);
        if (first + lane < KK) {
            delta = __builtin_fmaf(p, dp, delta);
            z += p;
            const uint32_t bits = __float_as_uint(fabsf(p * dp)), bits_p = __float_as_uint(p);
            most = most > bits ? most : bits;
            most_p = most_p > bits_p ? most_p : bits_p;
        }
        if (!kNormalised<T> && __ballot(delta != delta)) break;   // (fp32: part 2 needs the whole sum of the weights)
    }
    inv = kNormalised<T> ? 1.f / wave_sum(z) : 1.f;
    delta = wave_sum(delta) * inv;
    bound = ds_bound(__uint_as_float(wave_max(most)) * inv, __uint_as_float(wave_max(most_p)) * inv, delta);
    float acc[(D + kWave - 1) / kWave] = {};
    RasterWalk at;
    for (int first = 0; first < KK && delta == delta; first += kWave) {
        const int slot = first + lane < KK ? first + lane : KK - 1, a = slot / K, c = slot - a * K;
        float p, dp;
        pair_weight(m, g, scale, iy, ix, sy + a, sx + c, base, p, dp);
        const float ds = p * inv * (dp - delta);
        const int n = KK - first < kWave ? KK - first : kWave;
        for (int t = 0; t < n; ++t) {
            const float w = lane_value(ds, t);
#pragma unroll
            for (int u = 0; u < (D + kWave - 1) / kWave; ++u) {
                const int d = u * kWave + lane < D ? u * kWave + lane : D - 1;
                acc[u] = __builtin_fmaf(w, to_f32(m.k[((size_t)(sy + at.row) * g.W + sx + at.col) * D + d]), acc[u]);
            }
            at.next(K, K);
        }
    }
#pragma unroll
    for (int u = 0; u < (D + kWave - 1) / kWave; ++u)
        if (u * kWave + lane < D) replace_not_finite(dq + ((size_t)iy * g.W + ix) * D + u * kWave + lane, delta == delta ? scale * acc[u] : NAN);
    return delta;
}

// The kernel with two patches to a wave: the scale, that of its exponents, and what a query's products start from, -lse / scale rounded once.  (Where the start is
// off by a fraction of itself, every exponent of the query is off by that fraction of log2(e) lse.  Errors of dk and of the bias gradient against 64 bits over those of one patch to a
// wave, 90 x 26 x 27 fp16, k = 13: to logits of 440 1.00 to 1.01 and 1.00, of 1640 1.05 and 1.14, of 6600 1.05 and 1.20, from the sums' rounding at the start's size; with -1 / scale2 times
// log2(e) lse, three roundings, 1.06 and 1.05, 1.46 and 1.47, 1.51 and 1.58.)  A scale of 0 counts as 2^-100: what it adds to an exponent is 0 to fp32 for any |s| < 2^70.
__device__ __forceinline__ float start_scale(float scale) { return fabsf(scale) < 0x1p-100f ? __builtin_copysignf(0x1p-100f, scale) : scale; }
__device__ __forceinline__ float product_scale(float scale) { return start_scale(scale) * kLog2e; }
__device__ __forceinline__ float product_start(float lse, float scale, float inverse) {   // of start_scale(), and -1 over it
    const float x = lse * inverse;
    return fabsf(x) < INFINITY ? __builtin_fmaf(__builtin_fmaf(x, scale, lse), inverse, x) : x;
}

// dk and dv of one key from the queries that see it, likewise.
template <typename T, int D>
__device__ __forceinline__ void key_once_more(const PlanePtrs<T, D> &m, const PatchShape &g, float scale, int y, int x, const float *ld, T *dk, T *dv) {
    const int lane = threadIdx.x % kWave, K = g.K;
    const int y0 = inv_first(y, g.H, K), x0 = inv_first(x, g.W, K), nx = inv_last(x, g.W, K) - x0 + 1, ny = inv_last(y, g.H, K) - y0 + 1, total = ny * nx;
    constexpr int NU = (D + kWave - 1) / kWave;
    float ak[NU] = {}, av[NU] = {};
    RasterWalk at;
    for (int first = 0; first < total; first += kWave) {
        const int s = first + lane < total ? first + lane : total - 1, iy = y0 + s / nx, ix = x0 + s % nx;
        const size_t i_query = (size_t)iy * g.W + ix, plane_px = (size_t)g.H * g.W;
        const float *of = ld + (g.two ? 1 : kQueryWords<T>) * i_query;
        float p, dp;
        pair_weight(m, g, scale, iy, ix, y, x, g.two ? of[0] * -product_scale(scale) : of[0], p, dp);
        if constexpr (kNormalised<T>) p *= of[2];
        const float delta = g.two ? -of[plane_px] : of[1];
        const float ds = p * (dp - delta);
        const int n = total - first < kWave ? total - first : kWave;
        constexpr int kChunk = sizeof(T) == 4 ? 2 : 8;
        bool open = true;   // (a sum that is NaN stays NaN)
        for (int t0 = 0; t0 < n && open; t0 += kChunk) {
            float wp[kChunk], ws[kChunk], xd[kChunk][NU], xq[kChunk][NU];
#pragma unroll
            for (int e = 0; e < kChunk; ++e) {   // (their loads do not wait for each other; past the end: once more, not added)
                wp[e] = lane_value(p, (t0 + e) % kWave);
                ws[e] = lane_value(ds, (t0 + e) % kWave);
                const size_t i = ((size_t)(y0 + at.row) * g.W + x0 + at.col) * D;
                at.next(ny, nx);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int d = u * kWave + lane < D ? u * kWave + lane : D - 1;
                    xd[e][u] = to_f32(m.dout[i + d]);
                    xq[e][u] = to_f32(m.q[i + d]);
                }
            }
            bool any = false;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
#pragma unroll
                for (int e = 0; e < kChunk; ++e)
                    if (t0 + e < n) {
                        av[u] = __builtin_fmaf(wp[e], xd[e][u], av[u]);
                        ak[u] = __builtin_fmaf(ws[e], xq[e][u], ak[u]);
                    }
                any |= ak[u] == ak[u] || av[u] == av[u];
            }
            open = __ballot(any) != 0;
        }
        if (!open) break;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (u * kWave + lane < D) {
            const size_t o = ((size_t)y * g.W + x) * D + u * kWave + lane;
            replace_not_finite(dk + o, scale * ak[u]);
            replace_not_finite(dv + o, av[u]);
        }
}

// exp2(scale2 s + bias - base), bias in units of log2
template <typename T> __device__ __forceinline__ float exponential(float s, float scale2, float scale2_low, float bias, float base) {
    if constexpr (kNormalised<T>) return __builtin_amdgcn_exp2f(exponent_fp32(s, scale2, scale2_low, bias) - base);
    return __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s, bias - base));
}
template <typename T> __device__ __forceinline__ void store_query(float *ld, unsigned n, float base, float delta, float inv) {
    if constexpr (kNormalised<T>) *reinterpret_cast<f32x4 *>(ld + 4 * n) = f32x4{base, delta, inv, 0.f};
    else *reinterpret_cast<f32x2 *>(ld + 2 * n) = f32x2{base, delta};
}
// (ld: of the plane, of plane_px queries)
__device__ __forceinline__ void store_starts(float *ld, size_t plane_px, unsigned n, float start, float delta) {
    ld[n] = start;
    (ld + plane_px)[n] = -delta;
}

// What a query's dP are counted from, given its products with the values at the patch's 16 positions (in the layout of a block's products): their
// mean where it is larger than their spread, 0 otherwise (the mean of a few numbers around 0 would only add to the rounding).
// 2-norm error of dq against 64 bits at 8 x 2 x 40 x 40 queries, k = 13, values of unit variance and offsets per channel of variance 100, without / with
// it (the unfused steps): bf16 2.4e-2 / 2.6e-3 (1.7e-2), fp16 2.7e-3 / 3.2e-4 (1.9e-3), fp32 3.0e-6 / 8.6e-7 (1.6e-6); without offsets the same
// bits but for a few queries.  The pass takes 1 % longer (64 x 2 x 56 x 56, fp16, k = 13 277 / 280 us, fp32, k = 7 535 / 541; 64 channels 159 / 161).
__device__ __forceinline__ float near_mean(const f32x4 &near) {
    float sum = (near[0] + near[1]) + (near[2] + near[3]);
    float squares = __builtin_fmaf(near[0], near[0], near[1] * near[1]) + __builtin_fmaf(near[2], near[2], near[3] * near[3]);
    sum = column_sum(sum);
    squares = column_sum(squares);
    const float mean = sum * (1.f / 16.f);
    return mean * mean > squares * (1.f / 32.f) ? mean : 0.f;   // (what is not finite: 0)
}

// the lane's index, worked out anew
__device__ __forceinline__ int own_lane_index() {
    int zero = 0;
    asm volatile("" : "+v"(zero));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// ---- part 1 ------------------------------------------------------------------------------------------------------------
// ld: kQueryWords of every query, for part 2; bound: per query patch what no |dS| of the queries with a finite delta exceeds (bits of
// a float), and kMark where some delta is not finite; null where no bias gradient is wanted.
template <typename T, int D>
__global__ __launch_bounds__(kPatchThreads, (kPatchOcc<T, D>)) void patch_bwd_q_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale,
    const float *__restrict__ lse, const T *__restrict__ dout, T *__restrict__ dq, float *__restrict__ ld, uint32_t *__restrict__ bound, PatchShape g) {
    using CV = ChanVec<T, D>;
    using Op = PosOp<T, D>;
    constexpr int POSB = Op::POSB;
    extern __shared__ __align__(16) char lds[];
    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= g.units * g.splits) return;
    const WorkItem work = decode_work(wg, g.heads, g.tiles_y, g.splits, g.gd);
    const int head = work.head, K = g.K, H = g.H, W = g.W, NB = 2 * K - 1, pitch = bias_pitch(K);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int j = lane & 15, gr = lane >> 4;
    const int bias0 = dynamic_lds(lds), img0 = bias0 + bias_rows(K, g.with_bias) * pitch * 4;
    const int img_bytes = 4 * g.rw * POSB, stage_bytes = 2 * img_bytes;

    // a 4 x 4 patch per wave, 32 x 4, 16 x 8 or 8 x 16 positions per workgroup
    const int lg = g.lg_cols, tw = 4 << lg, th = 32 >> lg, ty0 = work.ty * th, tx0 = work.tx * tw;
    const int ty1 = ty0 + th - 1 < H - 1 ? ty0 + th - 1 : H - 1;
    const int ry0 = win_start(ty0, H, K), cx0 = win_start(tx0, W, K);            // first key row and column of the tile
    const int nsteps = (win_start(ty1, H, K) + K - ry0 + 3) >> 2;
    const int sy0 = ty0 + 4 * (wave >> lg), px0 = tx0 + 4 * (lg == 2 ? patch_of_wave(wave) : wave & ((1 << lg) - 1));   // this wave's patch
    const bool active = sy0 < H && px0 < W;
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1, px3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1;
    const int pyc = sy0 < H ? sy0 : H - 1, pxc = px0 < W ? px0 : W - 1;
    const int s_lo = (win_start(pyc, H, K) - ry0) >> 2, s_hi = (win_start(sy3, H, K) + K - 1 - ry0) >> 2;
    const int ox = win_start(pxc, W, K), nbx = (win_start(px3, W, K) + K - ox + 3) >> 2;
    const int qy = sy0 + (j >> 2), qx = px0 + (j & 3);
    const bool q_ok = qy < H && qx < W;
    const int iy = qy < H ? qy : H - 1, ix = qx < W ? qx : W - 1;
    const int wy = win_start(iy, H, K), wx = win_start(ix, W, K) - ox;           // window: first row, first column from ox
    const int aoff = ((j >> 2) * g.rw + (ox - cx0) + (j & 3)) * POSB + gr * CV::kLaneBytes;
    const int toff = Op::lane_offset(lane, g.rw) + (ox - cx0) * POSB;
    const int clear_lo = win_start(px3, W, K) - ox;   // columns [clear_lo, K) are in the window of every query of the patch
    const int u0 = ry0 + gr - iy + K - 1, boff = bias0 + (ox - ix + K - 1 + kBiasPad) * 4;
    const int no_row = boff + (bias_rows(K, g.with_bias) - 1) * pitch * 4;
    const size_t plane_px = (size_t)H * W;
    const int qlin = iy * W + ix;
    const float scale2 = scale * kLog2e, scale2_low = __builtin_fmaf(scale, kLog2e, -scale2) + scale * kLog2eLow;


    auto issue = [&](int b, int s, int par) {
        const size_t off = ((size_t)b * g.heads + head) * plane_px * POSB;
        const int img = img0 + par * stage_bytes;
        issue_rows<POSB>(reinterpret_cast<const char *>(k) + off, reinterpret_cast<const char *>(v) + off, H, W, ry0 + 4 * s, cx0, g.rw, img, img_bytes, wave, lane);
    };
    if (work.b_begin < work.b_end) issue(work.b_begin, 0, 0);
    stage_bias<T>(g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, K, g.by_pitch, bias0, tid);

    int par = 0;
    for (int b = work.b_begin; b < work.b_end; ++b) {
        const size_t plane = (size_t)b * g.heads + head;
        CV qo, dO;
        const size_t plane_off = plane * plane_px * POSB;
        // (a plane is smaller than 2^31 bytes: one 32-bit offset per lane for all tensors)
        qo.load(reinterpret_cast<const char *>(q) + plane_off + (unsigned)(qlin * POSB + gr * CV::kLaneBytes));
        dO.load(reinterpret_cast<const char *>(dout) + plane_off + (unsigned)(qlin * POSB + gr * CV::kLaneBytes));
        float base = (lse + plane * plane_px)[(unsigned)qlin] * kLog2e;
        if constexpr (kNormalised<T>) base = fabsf(base) < 32.f ? 0.f : __builtin_rintf(base);
        CV vo;
        vo.load(reinterpret_cast<const char *>(v) + plane_off + (unsigned)(qlin * POSB + gr * CV::kLaneBytes));
        settle(qo);
        settle(dO);
        settle(vo);
        const float from = near_mean(chan_dot<T, D>(vo, dO));
        const f32x4 less = sizeof(T) == 2 ? f32x4{-from, -from, -from, -from} : f32x4{0.f, 0.f, 0.f, 0.f};   // (fp32: subtracted below, for the registers)
        // sum of P dP k and of P k.  fp32: of a row of blocks at a time, then of the rows (one chain of K * K additions is off by twice as much)
        PosSum<T, D> sa, sp, row_a, row_p;
        sa.clear();
        sp.clear();
        if constexpr (sizeof(T) == 4) {
            row_a.clear();
            row_p.clear();
        }
        float delta = 0.f, most = 0.f, most_p = 0.f, z = 0.f;
        // N blocks of a row of blocks, from block column bx on
        auto blocks = [&](auto n, int img, int brow, int bx) {
            constexpr int N = decltype(n)::value;
            const int ka0 = img + aoff + bx * 4 * POSB, va0 = ka0 + img_bytes, kt0 = img + toff + bx * 4 * POSB, b0 = brow + bx * 16;
            CV ka[N], va[N];
            f32x4 sv[N], dp[N];
            Op kt[N];
            Weights4<T> wa[N], wp[N];
            float bias[N][4];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                ka[i].load_lds(ka0 + i * 4 * POSB);
                va[i].load_lds(va0 + i * 4 * POSB);
#pragma unroll
                for (int r = 0; r < 4; ++r) bias[i][r] = *lds_ptr<float>(b0 + i * 16 + r * 4);
                // columns outside the window: weight 0 (decided here: no branch may come between a product and the first use of its
                // result, see settle_products)
                if (4 * (bx + i) < clear_lo || 4 * (bx + i) + 4 > K) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) bias[i][r] = (unsigned)(4 * (bx + i) + r - wx) < (unsigned)K ? bias[i][r] : -INFINITY;
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                sv[i] = chan_dot<T, D>(ka[i], qo);
                dp[i] = chan_dot<T, D>(va[i], dO, less);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                kt[i].load_lds(kt0 + i * 4 * POSB);
                float p[4], w[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] = exponential<T>(sv[i][r], scale2, scale2_low, bias[i][r], base);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    w[r] = p[r] * (sizeof(T) == 4 ? dp[i][r] - from : dp[i][r]);
                    delta += w[r];
                    if constexpr (kNormalised<T>) z += p[r];
                    most = fmaxf(most, fabsf(w[r]));
                    most_p = fmaxf(most_p, p[r]);
                }
                wa[i] = Weights4<T>(w);
                wp[i] = Weights4<T>(p);
            }
            auto &ta = sizeof(T) == 4 ? row_a : sa, &tp = sizeof(T) == 4 ? row_p : sp;
            if constexpr (N == 2) {
                ta.add2(kt[0], wa[0], kt[1], wa[1]);
                tp.add2(kt[0], wp[0], kt[1], wp[1]);
            } else {
                if constexpr (kAtOnceQ<T, D> == 2) {
                    ta.add_last(kt[0], wa[0]);
                    tp.add_last(kt[0], wp[0]);
                } else {
                    ta.add(kt[0], wa[0]);
                    tp.add(kt[0], wp[0]);
                }
            }
        };
        for (int s = 0; s < nsteps; ++s) {
            wait_global_loads();
            workgroup_sync();   // this step's rows have landed for every wave, and nobody still reads the other buffer
            const int img = img0 + par * stage_bytes;
            const bool last = s + 1 == nsteps;
            if (g.nstage == 2) {
                par ^= 1;
                if (!last || b + 1 < work.b_end) issue(last ? b + 1 : b, last ? 0 : s + 1, par);
            }
            if (active && s >= s_lo && s <= s_hi) {
                const int u = u0 + 4 * s, uc = u < 0 ? 0 : (u < NB - 1 ? u : NB - 1);
                const bool rowok = (unsigned)(ry0 + 4 * s + gr - wy) < (unsigned)K;
                const int brow = rowok ? boff + (g.with_bias ? uc * pitch * 4 : 0) : no_row;
                constexpr int kAtOnce = kAtOnceQ<T, D>;
                int bx = 0;
                for (; bx + kAtOnce <= nbx; bx += kAtOnce) blocks(IntC<kAtOnce>{}, img, brow, bx);
                if (kAtOnce > 1 && bx < nbx) blocks(IntC<1>{}, img, brow, bx);
                if constexpr (sizeof(T) == 4) {
                    sa.take(row_a);
                    sp.take(row_p);
                }
            }
            if (g.nstage == 1 && (!last || b + 1 < work.b_end)) {
                workgroup_sync();   // nobody still reads the rows
                issue(last ? b + 1 : b, last ? 0 : s + 1, 0);
            }
        }
        if (!active) continue;
        if constexpr (sizeof(T) == 2) {
            sa.settle();
            sp.settle();
        }
        delta = column_sum(delta);
        float inv = 1.f;
        if constexpr (kNormalised<T>) {
            z = column_sum(z);
            inv = 1.f / z;
            delta *= inv;
        }
#pragma unroll
        for (int i = 0; i < Op::NA; ++i) sa.acc[i] -= delta * sp.acc[i];
        const float odd = __builtin_fmaf(delta, 0.f, sa.not_finite());   // NaN where something is not finite
        uint32_t bits = ds_bound(most * inv, most_p * inv, delta), mark = 0;   // (where delta is not finite: once more, below)
        if (q_ok) {
            sa.store(reinterpret_cast<char *>(dq) + plane_off, (unsigned)(qlin * POSB), gr, scale * inv);
            if (gr == 0) store_query<T>(ld + plane * plane_px * kQueryWords<T>, (unsigned)qlin, base, delta + from, inv);
        }
        unsigned long long again = __ballot(odd != odd);
        if (again) {
            wait_global_loads();   // (the stores above come first)
            PatchShape gc = g;     // (nothing of this is prepared outside of the branch)
            asm volatile("" : "+s"(gc.H), "+s"(gc.W), "+s"(gc.K));
            unsigned cols = (unsigned)((again | (again >> 16) | (again >> 32) | (again >> 48)) & 0xffffu);
            if ((cols >> j) & 1u) bits = 0;
            const PlanePtrs<T, D> m{q + plane * plane_px * D, k + plane * plane_px * D, v + plane * plane_px * D, dout + plane * plane_px * D,
                                    g.with_bias ? rpb + (size_t)head * NB * NB : nullptr};
            for (; cols; cols &= cols - 1) {
                const int c = __builtin_ctz(cols), cy = sy0 + (c >> 2), cx = px0 + (c & 3);
                if (cy >= H || cx >= W) continue;
                uint32_t own;
                float own_inv;
                const float b2 = lane_value(base, c);
                const float dl = query_once_more<T, D>(m, gc, scale, cy, cx, b2, dq + plane * plane_px * D, own, own_inv);
                if (lane == 0) store_query<T>(ld + plane * plane_px * kQueryWords<T>, (unsigned)(cy * W + cx), b2, dl, own_inv);
                if (own >= kNotFinite) mark = kMark;
                else bits = bits > own ? bits : own;
            }
        }
        if (bound != nullptr) {
            bits = wave_max(bits) | mark;
            if (lane == 0) bound[(plane * ((H + 3) >> 2) + (sy0 >> 2)) * ((W + 3) >> 2) + (px0 >> 2)] = bits;
        }
    }
}

// The end of a query patch of a plane for the kernel with two to a wave: delta, dq, what part 2 needs, and the bound of the patch; queries whose results are not finite once more.
template <typename T, int D>
__device__ __forceinline__ void finish_queries(PosSum<T, D> &sa, const PosSum<T, D> &sp, float delta, float most, float most_p, float start, float from, bool q_ok,
                                               int qlin, int lane, int sy0, int px0, size_t plane, int head, const T *q, const T *k, const T *v, const T *rpb, float scale,
                                               const T *dout, T *dq, float *ld, uint32_t *bound, const PatchShape &g) {
    using Op = PosOp<T, D>;
    const int H = g.H, W = g.W, NB = 2 * g.K - 1, j = lane & 15, gr = lane >> 4;
    const size_t plane_px = (size_t)H * W;
    delta = column_sum(delta);
#pragma unroll
    for (int i = 0; i < Op::NA; ++i) sa.acc[i] -= delta * sp.acc[i];
    const float odd = __builtin_fmaf(delta, 0.f, sa.not_finite());   // NaN where something is not finite
    uint32_t bits = q_ok ? ds_bound(most, most_p, delta) : 0, mark = 0;   // (where delta is not finite: once more, below)
    if (q_ok) {
        sa.store(reinterpret_cast<char *>(dq) + plane * plane_px * Op::POSB, (unsigned)(qlin * Op::POSB), gr, scale);
        if (gr == 0) store_starts(ld + plane * plane_px * kQueryWords<T>, plane_px, (unsigned)qlin, start, delta + from);
    }
    unsigned long long again = __ballot(odd != odd);
    if (again) {
        wait_global_loads();   // (the stores above come first)
        PatchShape gc = g;     // (nothing of this is prepared outside of the branch)
        asm volatile("" : "+s"(gc.H), "+s"(gc.W), "+s"(gc.K));
        unsigned cols = (unsigned)((again | (again >> 16) | (again >> 32) | (again >> 48)) & 0xffffu);
        if ((cols >> j) & 1u) bits = 0;
        const PlanePtrs<T, D> m{q + plane * plane_px * D, k + plane * plane_px * D, v + plane * plane_px * D, dout + plane * plane_px * D,
                                g.with_bias ? rpb + (size_t)head * NB * NB : nullptr};
        for (; cols; cols &= cols - 1) {
            const int c = __builtin_ctz(cols), cy = sy0 + (c >> 2), cx = px0 + (c & 3);
            if (cy >= H || cx >= W) continue;
            uint32_t own;
            float own_inv;
            const float s2 = lane_value(start, c);
            const float dl = query_once_more<T, D>(m, gc, scale, cy, cx, s2 * -product_scale(scale), dq + plane * plane_px * D, own, own_inv);
            if (lane == 0) store_starts(ld + plane * plane_px * kQueryWords<T>, plane_px, (unsigned)(cy * W + cx), s2, dl);
            if (own >= kNotFinite) mark = kMark;
            else bits = bits > own ? bits : own;
        }
    }
    if (bound != nullptr) {
        bits = wave_max(bits) | mark;
        if (lane == 0) bound[(plane * ((H + 3) >> 2) + (sy0 >> 2)) * ((W + 3) >> 2) + (px0 >> 2)] = bits;
    }
}

// Part 1 with two query patches to a wave, side by side (16 bit): they share the reads of the keys and values of a block and the bias row (the right
// one's is the left one's of the block before), as in part 2.  85 -> 78 us at 64 x 2 x 56 x 56 fp16, k = 13: 30 vector instructions per 16 x 16 products in the
// inner loop, as many again around it (a wave's prologue, its two patches' ends, the start of each row of blocks).
template <typename T, int D>
__global__ __launch_bounds__(kPatchThreads, 4) void patch_bwd_q2_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale,
    const float *__restrict__ lse, const T *__restrict__ dout, T *__restrict__ dq, float *__restrict__ ld, uint32_t *__restrict__ bound, PatchShape g) {
    static_assert(sizeof(T) == 2, "16 bit");
    using CV = ChanVec<T, D>;
    using Op = PosOp<T, D>;
    constexpr int POSB = Op::POSB;
    extern __shared__ __align__(16) char lds[];
    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= g.units * g.splits) return;
    const WorkItem work = decode_work(wg, g.heads, g.tiles_y, g.splits, g.gd);
    const int head = work.head, K = g.K, H = g.H, W = g.W, NB = 2 * K - 1, pitch = bias_pitch(K);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int bias0 = dynamic_lds(lds), img0 = bias0 + bias_rows(K, g.with_bias) * pitch * 4;
    const int img_bytes = 4 * g.rw * POSB, stage_bytes = 2 * img_bytes;

    const int lg = g.lg_cols, tw = 8 << lg, th = 32 >> lg, ty0 = work.ty * th, tx0 = work.tx * tw;
    const int ty1 = ty0 + th - 1 < H - 1 ? ty0 + th - 1 : H - 1;
    const int ry0 = win_start(ty0, H, K), cx0 = win_start(tx0, W, K);            // first key row and column of the tile
    const int nsteps = (win_start(ty1, H, K) + K - ry0 + 3) >> 2;
    const int sy0 = ty0 + 4 * (wave >> lg), px0 = tx0 + 8 * ((wave + 2 * (wave >> lg)) & ((1 << lg) - 1));   // this wave's left patch
    const bool active = sy0 < H && px0 < W, two = px0 + 4 < W;
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1, pyc = sy0 < H ? sy0 : H - 1;
    const int s_lo = (win_start(pyc, H, K) - ry0) >> 2, s_hi = (win_start(sy3, H, K) + K - 1 - ry0) >> 2;
    const int pl0 = px0 < W ? px0 : W - 1, pl3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1, pr0 = px0 + 4 < W - 1 ? px0 + 4 : W - 1, pr3 = px0 + 7 < W - 1 ? px0 + 7 : W - 1;
    // blocks of a row, counted from the left patch's first: the left patch's last, the right one's first and last
    const int ox = win_start(pl0, W, K), l_last = (win_start(pl3, W, K) + K - 1 - ox) >> 2;
    const int r_first = two ? (win_start(pr0, W, K) - ox) >> 2 : l_last + 1, r_last = two ? (win_start(pr3, W, K) + K - 1 - ox) >> 2 : l_last;
    // the first columns of the lane's windows; the columns that every query's window of a patch holds
    const int kx = px0 + (lane & 3);
    const int wx[2] = {win_start(kx < W ? kx : W - 1, W, K) - ox, win_start(kx + 4 < W ? kx + 4 : W - 1, W, K) - ox};
    const int clear_l0 = win_start(pl3, W, K) - ox, clear_l1 = K, clear_r0 = win_start(pr3, W, K) - ox, clear_r1 = win_start(pr0, W, K) + K - ox;
    const size_t plane_px = (size_t)H * W;
    const auto own_lane = own_lane_index;   // (recomputed where it is used: the registers)
    const auto query_of = [&](int lv, int right) {   // the lane's query of the left or the right patch, inside the map
        const int y = sy0 + ((lv & 15) >> 2), x = px0 + (lv & 3) + right;
        return (y < H - 1 ? y : H - 1) * W + (x < W - 1 ? x : W - 1);
    };
    const float scale2 = product_scale(scale), inverse = -1.f / start_scale(scale);

    auto issue = [&](int b, int s, int par) {
        const size_t off = ((size_t)b * g.heads + head) * plane_px * POSB;
        const int img = img0 + par * stage_bytes;
        issue_rows<POSB>(reinterpret_cast<const char *>(k) + off, reinterpret_cast<const char *>(v) + off, H, W, ry0 + 4 * s, cx0, g.rw, img, img_bytes, wave, lane);
    };
    if (work.b_begin < work.b_end) issue(work.b_begin, 0, 0);
    stage_bias<T>(g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, K, g.by_pitch, bias0, tid);

    int par = 0;
    for (int b = work.b_begin; b < work.b_end; ++b) {
        const size_t plane = (size_t)b * g.heads + head;
        CV qo[2], dO[2], vo[2];
        f32x4 from_s[2], from_dp[2];   // what the products start from
        const size_t plane_off = plane * plane_px * POSB;
        const int lv0 = own_lane();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // (a plane is smaller than 2^31 bytes: one 32-bit offset per lane for all tensors)
            const int at = query_of(lv0, 4 * t);
            const unsigned off = (unsigned)(at * POSB + (lv0 >> 4) * CV::kLaneBytes);
            qo[t].load(reinterpret_cast<const char *>(q) + plane_off + off);
            dO[t].load(reinterpret_cast<const char *>(dout) + plane_off + off);
            vo[t].load(reinterpret_cast<const char *>(v) + plane_off + off);
            from_s[t][0] = (lse + plane * plane_px)[(unsigned)at];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) settle(qo[t]), settle(dO[t]), settle(vo[t]);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float from = near_mean(chan_dot<T, D>(vo[t], dO[t])), s0 = product_start(from_s[t][0], start_scale(scale), inverse);
            from_s[t] = f32x4{s0, s0, s0, s0};
            from_dp[t] = f32x4{-from, -from, -from, -from};
        }
        PosSum<T, D> sa[2], sp[2];   // sum of P dP k and of P k
#pragma unroll
        for (int t = 0; t < 2; ++t) sa[t].clear(), sp[t].clear();
        float delta[2] = {0.f, 0.f}, most[2] = {0.f, 0.f}, most_p[2] = {0.f, 0.f};
        for (int s = 0; s < nsteps; ++s) {
            wait_global_loads();
            workgroup_sync();   // this step's rows have landed for every wave, and nobody still reads the other buffer
            const int img = img0 + par * stage_bytes;
            const bool last = s + 1 == nsteps;
            if (g.nstage == 2) {
                par ^= 1;
                if (!last || b + 1 < work.b_end) issue(last ? b + 1 : b, last ? 0 : s + 1, par);
            }
            if (active && s >= s_lo && s <= s_hi) {
                // the lane's queries' row against its row of the block (like its places in the images worked out anew in each step, for the registers)
                const int lv = own_lane(), j = lv & 15, gr = lv >> 4, x0 = ox - cx0;
                const int iy = sy0 + (j >> 2) < H - 1 ? sy0 + (j >> 2) : H - 1, krow = ry0 + 4 * s + gr;
                const bool rowok = (unsigned)(krow - win_start(iy, H, K)) < (unsigned)K;
                const int u = krow - iy + K - 1, uc = u < 0 ? 0 : (u < NB - 1 ? u : NB - 1);
                int brow = bias0 + ((rowok ? (g.with_bias ? uc : 0) : bias_rows(K, g.with_bias) - 1) * pitch + ox - px0 - (j & 3) + K - 1 + kBiasPad) * 4;
                int a0 = img + ((j >> 2) * g.rw + x0 + (j & 3)) * POSB + gr * CV::kLaneBytes, t0 = img + Op::lane_offset(lv, g.rw) + x0 * POSB;
                float before[4];   // the left patch's bias in the block before
                if (r_first == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) before[r] = *lds_ptr<float>(brow - 16 + r * 4);
                }
                // block column bx against the left patch (L), the right one (R) or both
                const auto block = [&](auto left, auto right, int bx) {
                    constexpr bool L = decltype(left)::value, R = decltype(right)::value;
                    CV ka, va;
                    ka.load_lds(a0);
                    va.load_lds(a0 + img_bytes);
                    float here[4], arg[2][4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (L) arg[0][r] = here[r] = *lds_ptr<float>(brow + r * 4);
                        if (R) arg[1][r] = L ? before[r] : *lds_ptr<float>(brow - 16 + r * 4);
                    }
                    // columns outside the window: weight 0 (decided before the products: no branch may come between one and the first use of its result,
                    // see settle_products)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        if (4 * bx < (t ? clear_r0 : clear_l0) || 4 * bx + 4 > (t ? clear_r1 : clear_l1)) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) arg[t][r] = (unsigned)(4 * bx + r - wx[t]) < (unsigned)K ? arg[t][r] : -INFINITY;
                        }
                    }
                    f32x4 s4[2], dp[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        s4[t] = chan_dot<T, D>(ka, qo[t], from_s[t]);
                        dp[t] = chan_dot<T, D>(va, dO[t], from_dp[t]);
                    }
                    Op kt;
                    kt.load_lds(t0);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        float p[4], w[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s4[t][r], arg[t][r]));
                            w[r] = p[r] * dp[t][r];
                            delta[t] += w[r];
                            most[t] = fmaxf(most[t], fabsf(w[r]));
                            most_p[t] = fmaxf(most_p[t], p[r]);
                        }
                        sa[t].add(kt, Weights4<T>(w));
                        sp[t].add(kt, Weights4<T>(p));
                    }
                    if (L) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) before[r] = here[r];
                    }
                    a0 += 4 * POSB;
                    t0 += 4 * POSB;
                    brow += 16;
                };
                int bx = 0;
                for (; bx < r_first; ++bx) block(IntC<1>{}, IntC<0>{}, bx);
                for (; bx <= l_last; ++bx) block(IntC<1>{}, IntC<1>{}, bx);
                for (; bx <= r_last; ++bx) block(IntC<0>{}, IntC<1>{}, bx);
            }
            if (g.nstage == 1 && (!last || b + 1 < work.b_end)) {
                workgroup_sync();   // nobody still reads the rows
                issue(last ? b + 1 : b, last ? 0 : s + 1, 0);
            }
        }
        if (!active) continue;
#pragma unroll
        for (int t = 0; t < 2; ++t) sa[t].settle(), sp[t].settle();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t == 1 && !two) continue;
            const int lv = own_lane(), qlin = query_of(lv, 4 * t);
            const bool q_ok = sy0 + ((lv & 15) >> 2) < H && px0 + (lv & 3) + 4 * t < W;
            finish_queries<T, D>(sa[t], sp[t], delta[t], most[t], most_p[t], from_s[t][0], -from_dp[t][0], q_ok, qlin, lv, sy0, px0 + 4 * t, plane, head, q, k, v, rpb, scale, dout, dq, ld, bound, g);
        }
    }
}

// ---- part 2 ------------------------------------------------------------------------------------------------------------
// What part 1 left of four map rows of queries for the kernel with two patches to a wave, rw from column x0 on, into LDS at `dst` by direct loads:
// 4 x rw starts, then as many -delta; a row each to the waves of a workgroup.  Positions outside the map as in issue_rows().
__device__ __forceinline__ void issue_starts(const float *ld, size_t plane_px, int H, int W, int y0, int x0, int rw, int dst, int wave, int lane) {
    asm volatile("" : "+s"(wave));   // (as in issue_rows)
    const int row = wave & 3, y = y0 + row < H - 1 ? y0 + row : H - 1;
    const char *from = reinterpret_cast<const char *>(ld + (wave >> 2 ? plane_px : 0));
    for (int s0 = 0; s0 < rw; s0 += kWave) {
        const int x = x0 + s0 + lane < W - 1 ? x0 + s0 + lane : W - 1;
        if (s0 + lane < rw) global_to_lds_4(from, (unsigned)((y * W + x) * 4), dst + (wave * rw + s0) * 4);
    }
}

// The bias gradient in LDS.  A plane's dS are added as integers dS 2^(kBits - E), 2^E bounding every |dS| that the workgroup
// meets in the plane (additions of integers commute, so waves may share the table); then the integers are added to the floating-point
// sums and cleared.  At most 256 keys of a tile add to a cell.  16 bit: 32-bit integers, a term rounded by 2^(E-24) at most, where
// the stored ds of the unfused steps is rounded at 2^-12 (fp16) of itself: error of the whole table against 64 bits 0.05 to 0.43 of theirs over 40 cases
// (k = 7 to 21, logits of unit and threefold scale, values and keys with and without offsets); the cells that only dS far below 2^E reach lose digits
// (99 % of the cells to 0.4 %, before to 1.5 to 200 %; with the threefold logits to 0.7 to 100 %, before to 13 to 140 %).
// fp32: 64-bit integers, rounded by 2^(E-51).
template <typename T> struct BiasSums {
    typedef int Int;
    typedef float Sum;
    static constexpr int kIntBytes = 4, kSumBytes = 4, kBits = 23;
    __device__ static __forceinline__ int to_int(float ds, float up) { return (int)__builtin_rintf(ds * up); }   // (a NaN counts as 0)
    __device__ static __forceinline__ void add_int(int addr, int n) { __hip_atomic_fetch_add(lds_ptr<int>(addr), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
    __device__ static __forceinline__ void add(int addr, float ds, float up) { add_int(addr, to_int(ds, up)); }
};
template <> struct BiasSums<float> {
    typedef long long Int;
    typedef double Sum;
    static constexpr int kIntBytes = 8, kSumBytes = 8, kBits = 50;
    __device__ static __forceinline__ void add(int addr, float ds, float up) {
        constexpr double kBig = 6755399441055744.0;   // 1.5 * 2^52: its mantissa's last bit counts 1
        const double x = __builtin_fma((double)(ds == ds ? ds : 0.f), (double)up, kBig);
        __hip_atomic_fetch_add(lds_ptr<long long>(addr), __builtin_bit_cast(long long, x) - __builtin_bit_cast(long long, kBig), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};
// Lanes of a wave whose offsets agree meet in one cell (row g of the block, row jy of the patch: jy - g), so each lane group has a
// copy of the integers of its own where the LDS holds four (copy g: the rows of its products start in banks that the other
// groups' do not use).
__host__ __device__ constexpr int int_words(int cells) { return (cells + 63) / 64 * 64 + 64; }   // per copy (integers)
__device__ __forceinline__ int copy_offset(int g, int cells) { return g * int_words(cells) + 8 * g + (g & 1) * 4 + (g >> 1) * 32; }
__host__ __device__ constexpr int flag_bytes(int cells) { return (cells + 127) / 128 * 16; }
template <typename T> __host__ __device__ constexpr int table_bytes(int cells, int copies) { return (copies > 1 ? copies * int_words(cells) : cells) * BiasSums<T>::kIntBytes; }
template <typename T> __host__ __device__ constexpr int dbias_bytes(int cells, int copies) { return cells * BiasSums<T>::kSumBytes + table_bytes<T>(cells, copies) + flag_bytes(cells); }

// The scale of a plane's integers, from the bounds of the query patches that the rectangle of queries touches (every wave finds the same): up = 2^(kBits - E),
// down its inverse; poisoned: some dS of the rectangle is not finite.
template <typename T>
__device__ __forceinline__ void bias_scale(const uint32_t *bound, size_t plane, int H, int W, int ry0, int cx0, int ry1, int cx1, int lane, float &up, float &down, bool &poisoned) {
    const int pw = (W + 3) >> 2, ph = (H + 3) >> 2, by0 = ry0 >> 2, bx0 = cx0 >> 2, bw = (cx1 >> 2) - bx0 + 1, nbound = ((ry1 >> 2) - by0 + 1) * bw;
    uint32_t most = 0, odd = 0;
    for (int i = lane; i < nbound; i += kWave) {
        const uint32_t bits = bound[(plane * ph + by0 + i / bw) * pw + bx0 + i % bw];
        odd |= bits & kMark;
        most = most > (bits & ~kMark) ? most : bits & ~kMark;
    }
    most = wave_max(most);
    poisoned = __ballot(odd != 0) != 0;
    int e = __builtin_amdgcn_readfirstlane((int)((most + 0x10000u) >> 23)) - 126;   // most < (1 - 2^-7) 2^e: 256 integers of kBits bits have a sum of 31
    e = e < -70 ? -70 : e;                                             // (2^(50 + 70) is a float)
    up = __builtin_ldexpf(1.f, BiasSums<T>::kBits - e);
    down = __builtin_ldexpf(1.f, e - BiasSums<T>::kBits);
}
// the integers of cell i, which are cleared
template <typename T> __device__ __forceinline__ typename BiasSums<T>::Int take_ints(int table0, int i, int cells, int copies) {
    typedef typename BiasSums<T>::Int Int;
    Int n = 0;
    for (int c = 0; c < copies; ++c) {
        const int a = table0 + ((c ? copy_offset(c, cells) : 0) + i) * (int)sizeof(Int);
        n += *lds_ptr<Int>(a);
        *lds_ptr<Int>(a) = 0;
    }
    return n;
}
// a workgroup's partial bias gradient (each thread reads the sums it added up)
template <typename T>
__device__ __forceinline__ void write_bias_sums(float *partial, int sums0, int flags0, const WorkItem &work, int head, int cells, int thread, const PatchShape &g) {
    const int NB = 2 * g.K - 1, pitch = bias_pitch(g.K);
    float *row = partial + (size_t)((head * g.splits + work.split) * g.gd.npos + work.pos) * rpb_cell_stride(NB * NB);
    for (int i = thread; i < cells; i += kPatchThreads) {
        const int u = fdiv(i, g.by_pitch), v = i - u * pitch - kBiasPad;
        if ((unsigned)v >= (unsigned)NB) continue;
        const bool odd = (*lds_ptr<unsigned>(flags0 + (i >> 5) * 4) >> (i & 31)) & 1u;
        row[u * NB + v] = odd ? NAN : (float)*lds_ptr<typename BiasSums<T>::Sum>(sums0 + i * BiasSums<T>::kSumBytes);
    }
}
// the keys of a patch (`again`: lanes) whose sums are not finite
template <typename T, int D>
__device__ __forceinline__ void keys_once_more(unsigned long long again, const T *q, const T *k, const T *v, const T *dout, const T *rpb, float scale, const float *ld, T *dk, T *dv,
                                               size_t plane, int head, int sy0, int px0, const PatchShape &g) {
    wait_global_loads();   // (the stores come first)
    PatchShape gc = g;     // (nothing of this is prepared outside of the branch)
    asm volatile("" : "+s"(gc.H), "+s"(gc.W), "+s"(gc.K));
    const int NB = 2 * g.K - 1;
    const size_t px = (size_t)g.H * g.W, at = plane * px * D;
    const PlanePtrs<T, D> m{q + at, k + at, v + at, dout + at, g.with_bias ? rpb + (size_t)head * NB * NB : nullptr};
    for (unsigned cols = (unsigned)((again | (again >> 16) | (again >> 32) | (again >> 48)) & 0xffffu); cols; cols &= cols - 1) {
        const int c = __builtin_ctz(cols), cy = sy0 + (c >> 2), cx = px0 + (c & 3);
        if (cy < g.H && cx < g.W) key_once_more<T, D>(m, gc, scale, cy, cx, ld + kQueryWords<T> * plane * px, dk + at, dv + at);
    }
}

// LGS 1: two waves share a patch, the even and the odd rows of blocks, and a workgroup takes one plane (its integers go straight to its partial
// bias gradient).
template <typename T, int D, int LGS>
__global__ __launch_bounds__(kPatchThreads, (kPatchOcc<T, D>)) void patch_bwd_kv_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale,
    const float *__restrict__ ld, const uint32_t *__restrict__ bound, const T *__restrict__ dout, T *__restrict__ dk, T *__restrict__ dv,
    float *__restrict__ partial, PatchShape g) {
    using CV = ChanVec<T, D>;
    using Op = PosOp<T, D>;
    constexpr int POSB = Op::POSB, QB = kQueryWords<T> * 4, STEP = 4 << LGS;   // map rows per step
    extern __shared__ __align__(16) char lds[];
    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= g.units * g.splits) return;
    const WorkItem work = decode_work(wg, g.heads, g.tiles_y, g.splits, g.gd);
    const int head = work.head, K = g.K, H = g.H, W = g.W, NB = 2 * K - 1, pitch = bias_pitch(K);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int j = lane & 15, gr = lane >> 4;
    const int part = wave & ((1 << LGS) - 1), pw = wave >> LGS;   // the wave's row of blocks in a step, and its patch of the tile
    using Table = BiasSums<T>;
    const int cells = NB * pitch, sums0 = dynamic_lds(lds), table0 = sums0 + (g.with_dbias && LGS == 0 ? cells * Table::kSumBytes : 0);
    const int flags0 = table0 + (g.with_dbias ? table_bytes<T>(cells, g.copies) : 0), bias0 = flags0 + (g.with_dbias ? flag_bytes(cells) : 0);
    const int img0 = bias0 + bias_rows(K, g.with_bias) * pitch * 4;
    const int img_bytes = STEP * g.rw * POSB, stage_bytes = 2 * img_bytes + STEP * g.rw * QB;

    const int lg = g.lg_cols, tw = 4 << lg, th = (32 >> LGS) >> lg, ty0 = work.ty * th, tx0 = work.tx * tw;
    const int ty1 = ty0 + th - 1 < H - 1 ? ty0 + th - 1 : H - 1, tx1 = tx0 + tw - 1 < W - 1 ? tx0 + tw - 1 : W - 1;
    const int ry0 = inv_first(ty0, H, K), cx0 = inv_first(tx0, W, K);            // first query row and column of the tile
    const int ry1 = inv_last(ty1, H, K), cx1 = inv_last(tx1, W, K);
    const int nsteps = (ry1 - ry0 + STEP) >> (2 + LGS);
    const int sy0 = ty0 + 4 * (pw >> lg), px0 = tx0 + 4 * (lg == 2 && LGS == 0 ? patch_of_wave(pw) : pw & ((1 << lg) - 1));   // this wave's patch
    const bool active = sy0 < H && px0 < W;
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1, px3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1;
    const int pyc = sy0 < H ? sy0 : H - 1, pxc = px0 < W ? px0 : W - 1;
    const int b_lo = (inv_first(pyc, H, K) - ry0) >> 2, b_hi = (inv_last(sy3, H, K) - ry0) >> 2;   // rows of blocks
    const int ox = inv_first(pxc, W, K), nbx = (inv_last(px3, W, K) - ox + 4) >> 2;
    const int ky = sy0 + (j >> 2), kx = px0 + (j & 3);
    const bool key_ok = ky < H && kx < W;
    const int jx = kx < W ? kx : W - 1;
    // the columns of the queries that see the lane's key: the first (from ox) and their number
    const int fx = inv_first(jx, W, K) - ox, nx = inv_last(jx, W, K) - ox - fx + 1;
    const int aoff = ((4 * part + (j >> 2)) * g.rw + (ox - cx0) + (j & 3)) * POSB + gr * CV::kLaneBytes;
    const int toff = Op::lane_offset(lane, g.rw) + (4 * part * g.rw + ox - cx0) * POSB;
    // columns [clear_lo, clear_hi) see every key of the patch
    const int clear_lo = inv_first(px3, W, K) - ox, clear_hi = inv_last(pxc, W, K) + 1 - ox, no_row = bias_rows(K, g.with_bias) - 1;
    const int loff = ((4 * part + gr) * g.rw + (ox - cx0)) * QB;
    const int v0 = jx - ox + K - 1 + kBiasPad;     // (the cell falls with the query's row and column)
    const size_t plane_px = (size_t)H * W;
    const auto own_lane = own_lane_index;   // (recomputed where it is used: a register less in the inner loop)
    const auto key_offset = [&](int lv) {
        const int y = sy0 + ((lv & 15) >> 2), x = px0 + (lv & 3);
        return (unsigned)(((y < H - 1 ? y : H - 1) * W + (x < W - 1 ? x : W - 1)) * POSB);
    };
    const int table_lane = table0 + (g.copies > 1 ? copy_offset(gr, cells) * Table::kIntBytes : 0);
    const float scale2 = scale * kLog2e, scale2_low = __builtin_fmaf(scale, kLog2e, -scale2) + scale * kLog2eLow;

    auto issue = [&](int b, int s, int par) {
        const size_t px = ((size_t)b * g.heads + head) * plane_px;
        const int img = img0 + par * stage_bytes;
        issue_rows<POSB>(reinterpret_cast<const char *>(q) + px * POSB, reinterpret_cast<const char *>(dout) + px * POSB, H, W, ry0 + STEP * s, cx0, g.rw, img, img_bytes, wave, lane, STEP);
        int w = wave;
        asm volatile("" : "+s"(w));
        const int row = w & (STEP - 1), y = ry0 + STEP * s + row < H - 1 ? ry0 + STEP * s + row : H - 1;
        constexpr int LB = kNormalised<T> ? 16 : 4, PER = QB / LB;   // bytes a lane loads, lanes per query
        for (int s0 = (w >> (2 + LGS)) * kWave; s0 < PER * g.rw; s0 += (kPatchWaves / STEP) * kWave) {
            const int c = s0 + lane;
            int x = cx0 + c / PER;
            x = x < W - 1 ? x : W - 1;
            const unsigned off = (unsigned)((y * W + x) * QB + (c % PER) * LB);
            const int dst = img + 2 * img_bytes + row * g.rw * QB + s0 * LB;
            if (c < PER * g.rw) {
                if constexpr (LB == 16) global_to_lds_16(reinterpret_cast<const char *>(ld) + px * QB, off, dst);
                else global_to_lds_4(reinterpret_cast<const char *>(ld) + px * QB, off, dst);
            }
        }
    };
    if (work.b_begin < work.b_end) issue(work.b_begin, 0, 0);
    stage_bias<T>(g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, K, g.by_pitch, bias0, tid);
    if (g.with_dbias)
        for (int i = sums0 + tid * 16; i < bias0; i += kPatchThreads * 16) *lds_ptr<u32x4>(i) = u32x4{0u, 0u, 0u, 0u};

    int par = 0;
    for (int b = work.b_begin; b < work.b_end; ++b) {
        const size_t plane = (size_t)b * g.heads + head;
        CV ko, vo;
        const size_t plane_off = plane * plane_px * POSB;
        const int lv0 = own_lane();
        const unsigned key_lane = key_offset(lv0) + (lv0 >> 4) * CV::kLaneBytes;
        ko.load(reinterpret_cast<const char *>(k) + plane_off + key_lane);
        vo.load(reinterpret_cast<const char *>(v) + plane_off + key_lane);
        settle(ko);
        settle(vo);
        float up = 0.f, down = 0.f;   // 2^(kBits - E) and its inverse
        bool poisoned = false;  // some dS of the plane's rectangle is not finite
        if (g.with_dbias) bias_scale<T>(bound, plane, H, W, ry0, cx0, ry1, cx1, own_lane(), up, down, poisoned);
        PosSum<T, D> sk, sv, row_k, row_v;   // (fp32: of a row of blocks, then of the rows, as in part 1)
        sk.clear();
        sv.clear();
        if constexpr (sizeof(T) == 4) {
            row_k.clear();
            row_v.clear();
        }
        // N blocks of a row of blocks, from block column bx on
        auto blocks = [&](auto n, int img, int brow, int cell, bool rowok, int bx) {
            constexpr int N = decltype(n)::value;
            const int qa0 = img + aoff + bx * 4 * POSB, da0 = qa0 + img_bytes, qt0 = img + toff + bx * 4 * POSB, dt0 = qt0 + img_bytes;
            constexpr bool kTight = sizeof(T) == 4 && D == 32;   // (16 bit has the registers: 2 % faster with all of a block's reads in flight)
            const int l0 = img + 2 * img_bytes + loff + bx * 4 * QB, b0 = brow - bx * 16, c0 = cell - 4 * bx;
            f32x4 s4[N], dp[N];
            Weights4<T> wp[N], ws[N];
            typedef float Of __attribute__((ext_vector_type(kNormalised<T> ? 3 : 2)));
            Of l[N][4];   // what part 1 left of the queries
            float bias[N][4];
            CV qa[N], da[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if constexpr (!kTight) {
                    qa[i].load_lds(qa0 + i * 4 * POSB);
                    da[i].load_lds(da0 + i * 4 * POSB);
                }
                if constexpr (sizeof(T) == 2) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) bias[i][r] = *lds_ptr<float>(b0 - i * 16 - r * 4);
                    // queries whose windows do not hold the key: weight 0 (decided before the products, as in part 1)
                    if (4 * (bx + i) < clear_lo || 4 * (bx + i) + 4 > clear_hi) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) bias[i][r] = (unsigned)(4 * (bx + i) + r - fx) < (unsigned)nx ? bias[i][r] : -INFINITY;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if constexpr (kTight) qa[i].load_lds(qa0 + i * 4 * POSB);
                s4[i] = chan_dot<T, D>(qa[i], ko);
                if constexpr (kTight && sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);   // (not all loads at once: the registers)
                if constexpr (kTight) da[i].load_lds(da0 + i * 4 * POSB);
                dp[i] = chan_dot<T, D>(da[i], vo);
                if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    l[i][r] = *lds_ptr<Of>(l0 + (4 * i + r) * QB);
                    // (fp32, bound by the matrix cores: every block is masked, and the bias comes late, for the registers)
                    if constexpr (sizeof(T) == 4) {
                        const float t = *lds_ptr<float>(b0 - i * 16 - r * 4);
                        bias[i][r] = (unsigned)(4 * (bx + i) + r - fx) < (unsigned)nx ? t : -INFINITY;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
                float p[4], ds[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[r] = exponential<T>(s4[i][r], scale2, scale2_low, bias[i][r], l[i][r].x);
                    if constexpr (kNormalised<T>) p[r] *= l[i][r].z;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) ds[r] = p[r] * (dp[i][r] - l[i][r].y);
                if (g.with_dbias) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) Table::add(table_lane + (c0 - 4 * i - r) * Table::kIntBytes, ds[r], up);   // (outside the window: 0)
                    if (poisoned) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int c = c0 - 4 * i - r;
                            const bool in = rowok && (unsigned)(4 * (bx + i) + r - fx) < (unsigned)nx;
                            if (in && !(fabsf(ds[r]) < INFINITY)) __hip_atomic_fetch_or(lds_ptr<unsigned>(flags0 + (c >> 5) * 4), 1u << (c & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                }
                wp[i] = Weights4<T>(p);
                ws[i] = Weights4<T>(ds);
            }
            if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
            Op t[N];
#pragma unroll
            for (int i = 0; i < N; ++i) t[i].load_lds(dt0 + i * 4 * POSB);
            auto &tk = sizeof(T) == 4 ? row_k : sk, &tv = sizeof(T) == 4 ? row_v : sv;
            if constexpr (N == 2) tv.add2(t[0], wp[0], t[1], wp[1]);
            else if constexpr (kAtOnceKv<T, D> == 2) tv.add_last(t[0], wp[0]);
            else tv.add(t[0], wp[0]);
            if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < N; ++i) t[i].load_lds(qt0 + i * 4 * POSB);
            if constexpr (N == 2) tk.add2(t[0], ws[0], t[1], ws[1]);
            else if constexpr (kAtOnceKv<T, D> == 2) tk.add_last(t[0], ws[0]);
            else tk.add(t[0], ws[0]);
        };
        for (int s = 0; s < nsteps; ++s) {
            wait_global_loads();
            workgroup_sync();   // this step's rows have landed for every wave, and nobody still reads the other buffer
            const int img = img0 + par * stage_bytes;
            const bool last = s + 1 == nsteps;
            if (g.nstage == 2) {
                par ^= 1;
                if (!last || b + 1 < work.b_end) issue(last ? b + 1 : b, last ? 0 : s + 1, par);
            }
            const int br = (s << LGS) + part;   // this wave's row of blocks
            if (active && br >= b_lo && br <= b_hi) {
                // the lane's row of the block against its key (fp32: worked out anew in each step, for the registers)
                const int lv = sizeof(T) == 4 ? own_lane_index() : lane;
                const int qrow = ry0 + 4 * br + (lv >> 4), krow = sy0 + ((lv & 15) >> 2), kc = krow < H ? krow : H - 1, first = inv_first(kc, H, K);
                const bool rowok = krow < H && px0 + (lv & 3) < W && qrow >= first && qrow <= inv_last(kc, H, K);
                const int u = kc - qrow + K - 1, uc = u < 0 ? 0 : (u < NB - 1 ? u : NB - 1);
                const int cell = uc * pitch + v0, brow = bias0 + ((rowok ? (g.with_bias ? uc : 0) : no_row) * pitch + v0) * 4;
                constexpr int kAtOnce = kAtOnceKv<T, D>;
                int bx = 0;
                for (; bx + kAtOnce <= nbx; bx += kAtOnce) blocks(IntC<kAtOnce>{}, img, brow, cell, rowok, bx);
                if (kAtOnce > 1 && bx < nbx) blocks(IntC<1>{}, img, brow, cell, rowok, bx);
                if constexpr (sizeof(T) == 4) {
                    sk.take(row_k);
                    sv.take(row_v);
                }
            }
            if (g.nstage == 1 && (!last || b + 1 < work.b_end)) {
                workgroup_sync();   // nobody still reads the rows
                issue(last ? b + 1 : b, last ? 0 : s + 1, 0);
            }
        }
        if constexpr (sizeof(T) == 2) {
            sk.settle();
            sv.settle();
        }
        if (g.with_dbias) {
            workgroup_sync();   // every wave has added its part; nobody adds more before the next step's barrier
            for (int i = wave * kWave + own_lane(); i < cells; i += kPatchThreads) {
                const typename Table::Int n = take_ints<T>(table0, i, cells, g.copies);
                if constexpr (LGS > 0) {
                    const int u = fdiv(i, g.by_pitch), v = i - u * pitch - kBiasPad;
                    if ((unsigned)v < (unsigned)NB) {
                        const bool odd = (*lds_ptr<unsigned>(flags0 + (i >> 5) * 4) >> (i & 31)) & 1u;
                        partial[(size_t)((head * g.splits + work.split) * g.gd.npos + work.pos) * rpb_cell_stride(NB * NB) + u * NB + v] =
                            odd ? NAN : (float)((typename Table::Sum)n * (typename Table::Sum)down);
                    }
                } else {
                    *lds_ptr<typename Table::Sum>(sums0 + i * Table::kSumBytes) += (typename Table::Sum)n * (typename Table::Sum)down;
                }
            }
        }
        if constexpr (LGS > 0) {
            // the two waves of a patch, joined by the first (one plane per workgroup: nothing is on its way to the images)
            static_assert(LGS == 1 && sizeof(T) == 2, "pairs of waves");
            workgroup_sync();
            const int mine = img0 + pw * Op::NA * 2048 + lane * 16;
            if (part > 0) {
#pragma unroll
                for (int i = 0; i < Op::NA; ++i) {
                    *lds_ptr<f32x4>(mine + i * 2048) = sk.acc[i];
                    *lds_ptr<f32x4>(mine + i * 2048 + 1024) = sv.acc[i];
                }
            }
            workgroup_sync();
            if (part > 0) continue;
#pragma unroll
            for (int i = 0; i < Op::NA; ++i) {
                sk.acc[i] += *lds_ptr<f32x4>(mine + i * 2048);
                sv.acc[i] += *lds_ptr<f32x4>(mine + i * 2048 + 1024);
            }
        }
        if (!active) continue;
        if (key_ok) {
            const int lv = own_lane();
            const unsigned o = key_offset(lv);
            sk.store(reinterpret_cast<char *>(dk) + plane_off, o, lv >> 4, scale);
            sv.store(reinterpret_cast<char *>(dv) + plane_off, o, lv >> 4, 1.f);
        }
        const float odd = sk.not_finite() + sv.not_finite();
        const unsigned long long again = __ballot(odd != odd);
        if (again) keys_once_more<T, D>(again, q, k, v, dout, rpb, scale, ld, dk, dv, plane, head, sy0, px0, g);
    }
    if (LGS == 0 && g.with_dbias) write_bias_sums<T>(partial, sums0, flags0, work, head, cells, wave * kWave + own_lane(), g);
}

// Part 2 with two key patches to a wave, side by side (16 bit).  The left patch meets a block of queries in the cells of the bias table in which the
// right one meets the next block: the two share the reads of the queries, upstream gradients, starts and deltas of a block, the bias row (the
// right one's is the left one's of the block before) and the integer additions (likewise), and half as many rows of blocks are walked.  That, products that
// start from -lse / scale and -delta, and no branch between the results of the two: vector instructions of the kernel 49e6 -> 39e6 at 64 x 2 x 56 x 56 fp16, k = 13,
// 146 -> 118 us.  It is bound by their issue (in a full round three quarters of the slots; a wave's prologue and the barrier of each step, where
// the waves next to a border have up to half as many blocks more, are the rest).
template <typename T, int D, bool DBIAS>
__global__ __launch_bounds__(kPatchThreads, 4) void patch_bwd_kv2_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale,
    const float *__restrict__ ld, const uint32_t *__restrict__ bound, const T *__restrict__ dout, T *__restrict__ dk, T *__restrict__ dv,
    float *__restrict__ partial, PatchShape g) {
    static_assert(sizeof(T) == 2, "16 bit");
    using CV = ChanVec<T, D>;
    using Op = PosOp<T, D>;
    using Table = BiasSums<T>;
    constexpr int POSB = Op::POSB;
    extern __shared__ __align__(16) char lds[];
    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= g.units * g.splits) return;
    const WorkItem work = decode_work(wg, g.heads, g.tiles_y, g.splits, g.gd);
    const int head = work.head, K = g.K, H = g.H, W = g.W, NB = 2 * K - 1, pitch = bias_pitch(K);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int cells = NB * pitch, sums0 = dynamic_lds(lds), table0 = sums0 + (DBIAS ? cells * Table::kSumBytes : 0);
    const int flags0 = table0 + (DBIAS ? table_bytes<T>(cells, g.copies) : 0), bias0 = flags0 + (DBIAS ? flag_bytes(cells) : 0);
    const int img0 = bias0 + bias_rows(K, g.with_bias) * pitch * 4;
    const int img_bytes = 4 * g.rw * POSB, ld_bytes = 16 * g.rw, stage_bytes = 2 * img_bytes + 2 * ld_bytes;

    const int lg = g.lg_cols, tw = 8 << lg, th = 32 >> lg, ty0 = work.ty * th, tx0 = work.tx * tw;
    const int ty1 = ty0 + th - 1 < H - 1 ? ty0 + th - 1 : H - 1, tx1 = tx0 + tw - 1 < W - 1 ? tx0 + tw - 1 : W - 1;
    const int ry0 = inv_first(ty0, H, K), cx0 = inv_first(tx0, W, K);            // first query row and column of the tile
    const int ry1 = inv_last(ty1, H, K), cx1 = inv_last(tx1, W, K);
    const int nsteps = (ry1 - ry0 + 4) >> 2;
    
    // this wave's left patch: the lower rows of pairs are taken in another order, so that the waves of a SIMD (w and w + 4) do not all get those
    // next to a border, which meet up to half as many blocks more
    const int sy0 = ty0 + 4 * (wave >> lg), px0 = tx0 + 8 * ((wave + 2 * (wave >> lg)) & ((1 << lg) - 1));
    const bool active = sy0 < H && px0 < W, two = px0 + 4 < W;
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1;
    const int pyc = sy0 < H ? sy0 : H - 1;
    const int b_lo = (inv_first(pyc, H, K) - ry0) >> 2, b_hi = (inv_last(sy3, H, K) - ry0) >> 2;   // rows of blocks
    const int pl0 = px0 < W ? px0 : W - 1, pl3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1, pr0 = px0 + 4 < W - 1 ? px0 + 4 : W - 1, pr3 = px0 + 7 < W - 1 ? px0 + 7 : W - 1;
    // blocks of a row, counted from the left patch's first: the left patch's last, the right one's first and last
    const int ox = inv_first(pl0, W, K), l_last = (inv_last(pl3, W, K) - ox) >> 2;
    const int r_first = two ? (inv_first(pr0, W, K) - ox) >> 2 : l_last + 1, r_last = two ? (inv_last(pr3, W, K) - ox) >> 2 : l_last;
    // the columns of the queries that see the lane's keys: the first (from ox) and their number (0: a key outside the map)
    const int kx = px0 + (lane & 3), kl = kx < W ? kx : W - 1, kr = kx + 4 < W ? kx + 4 : W - 1;
    const auto span = [&](int x, int kc) { return (inv_first(kc, W, K) - ox) | ((x < W ? inv_last(kc, W, K) - inv_first(kc, W, K) + 1 : 0) << 16); };   // (below 2^15, two to a register)
    const int spans[2] = {span(kx, kl), span(kx + 4, kr)};
    // columns that see every key of a patch
    const int clear_l0 = inv_first(pl3, W, K) - ox, clear_l1 = px0 + 3 < W ? inv_last(pl0, W, K) + 1 - ox : 0;
    const int clear_r0 = inv_first(pr3, W, K) - ox, clear_r1 = px0 + 7 < W ? inv_last(pr0, W, K) + 1 - ox : 0;
    const int no_row = bias_rows(K, g.with_bias) - 1;
    const size_t plane_px = (size_t)H * W;
    const auto own_lane = own_lane_index;   // (recomputed where it is used: a register less in the inner loop)
    const auto key_offset = [&](int lv, int right) {
        const int y = sy0 + ((lv & 15) >> 2), x = px0 + (lv & 3) + right;
        return (unsigned)(((y < H - 1 ? y : H - 1) * W + (x < W - 1 ? x : W - 1)) * POSB);
    };
    const float scale2 = product_scale(scale);

    auto issue = [&](int b, int s, int par) {
        const size_t px = ((size_t)b * g.heads + head) * plane_px;
        const int img = img0 + par * stage_bytes;
        issue_rows<POSB>(reinterpret_cast<const char *>(q) + px * POSB, reinterpret_cast<const char *>(dout) + px * POSB, H, W, ry0 + 4 * s, cx0, g.rw, img, img_bytes, wave, lane);
        issue_starts(ld + px * kQueryWords<T>, plane_px, H, W, ry0 + 4 * s, cx0, g.rw, img + 2 * img_bytes, wave, lane);
    };
    if (work.b_begin < work.b_end) issue(work.b_begin, 0, 0);
    stage_bias<T>(g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, K, g.by_pitch, bias0, tid);
    if (DBIAS)
        for (int i = sums0 + tid * 16; i < bias0; i += kPatchThreads * 16) *lds_ptr<u32x4>(i) = u32x4{0u, 0u, 0u, 0u};

    int par = 0;
    for (int b = work.b_begin; b < work.b_end; ++b) {
        const size_t plane = (size_t)b * g.heads + head;
        CV ko[2], vo[2];
        const size_t plane_off = plane * plane_px * POSB;
        const int lv0 = own_lane();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const unsigned key_lane = key_offset(lv0, 4 * t) + (lv0 >> 4) * CV::kLaneBytes;
            ko[t].load(reinterpret_cast<const char *>(k) + plane_off + key_lane);
            vo[t].load(reinterpret_cast<const char *>(v) + plane_off + key_lane);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) settle(ko[t]), settle(vo[t]);
        float up = 0.f, down = 0.f;   // 2^(kBits - E) and its inverse
        bool poisoned = false;  // some dS of the plane's rectangle is not finite
        if (DBIAS) bias_scale<T>(bound, plane, H, W, ry0, cx0, ry1, cx1, own_lane(), up, down, poisoned);
        PosSum<T, D> sk[2], sv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) sk[t].clear(), sv[t].clear();
        for (int s = 0; s < nsteps; ++s) {
            wait_global_loads();
            workgroup_sync();   // this step's rows have landed for every wave, and nobody still reads the other buffer
            const int img = img0 + par * stage_bytes;
            const bool last = s + 1 == nsteps;
            if (g.nstage == 2) {
                par ^= 1;
                if (!last || b + 1 < work.b_end) issue(last ? b + 1 : b, last ? 0 : s + 1, par);
            }
            if (active && s >= b_lo && s <= b_hi) {
                // the lane's row of the block against its keys' row (like the lane's places in the images worked out anew in each step, for the registers)
                const int lv = own_lane(), j = lv & 15, gr = lv >> 4, x0 = ox - cx0;
                const int table_lane = table0 + (g.copies > 1 ? copy_offset(gr, cells) * Table::kIntBytes : 0);
                const int v0 = px0 + (j & 3) - ox + K - 1 + kBiasPad;     // (the cell falls with the query's row and column)
                const int qrow = ry0 + 4 * s + gr, krow = sy0 + (j >> 2), kc = krow < H ? krow : H - 1, first = inv_first(kc, H, K);
                const bool rowok = krow < H && qrow >= first && qrow <= inv_last(kc, H, K);
                const int u = kc - qrow + K - 1, uc = u < 0 ? 0 : (u < NB - 1 ? u : NB - 1);
                int cell = table_lane + (uc * pitch + v0) * 4, brow = bias0 + ((rowok ? (g.with_bias ? uc : 0) : no_row) * pitch + v0) * 4 - 12;   // (of the last of four columns)
                int a0 = img + ((j >> 2) * g.rw + x0 + (j & 3)) * POSB + gr * CV::kLaneBytes, t0 = img + Op::lane_offset(lv, g.rw) + x0 * POSB;
                int l0 = img + 2 * img_bytes + (gr * g.rw + x0) * 4;
                float before[4];   // the left patch's bias in the block before
                int held[4];       // and its dS there
#pragma unroll
                for (int r = 0; r < 4; ++r) held[r] = 0;
                if (r_first == 0) {
#pragma unroll
                    for (int r = 3; r >= 0; --r) before[r] = *lds_ptr<float>(brow + 28 - r * 4);
                }
                // block column bx against the left patch (L), the right one (R) or both
                const auto block = [&](auto left, auto right, int bx) {
                    constexpr bool L = decltype(left)::value, R = decltype(right)::value;
                    CV qa, da;
                    qa.load_lds(a0);
                    da.load_lds(a0 + img_bytes);
                    f32x4 from_s, from_dp;
                    float here[4], arg[2][4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        from_s[r] = *lds_ptr<float>(l0 + r * 4);
                        from_dp[r] = *lds_ptr<float>(l0 + ld_bytes + r * 4);
                    }
#pragma unroll
                    for (int r = 3; r >= 0; --r) {
                        if (L) arg[0][r] = here[r] = *lds_ptr<float>(brow + 12 - r * 4);
                        if (R) arg[1][r] = L ? before[r] : *lds_ptr<float>(brow + 28 - r * 4);
                    }
                    // queries whose windows do not hold the key: weight 0 (decided before the products, as in part 1)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        if (4 * bx < (t ? clear_r0 : clear_l0) || 4 * bx + 4 > (t ? clear_r1 : clear_l1)) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) arg[t][r] = (unsigned)(4 * bx + r - (spans[t] & 0xffff)) < (unsigned)spans[t] >> 16 ? arg[t][r] : -INFINITY;
                        }
                    }
                    f32x4 s4[2], dp[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        s4[t] = chan_dot<T, D>(qa, ko[t], from_s);
                        dp[t] = chan_dot<T, D>(da, vo[t], from_dp);
                    }
                    Op qt, dt;
                    dt.load_lds(t0 + img_bytes);
                    qt.load_lds(t0);
                    float p[2][4], ds[2][4];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            p[t][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s4[t][r], arg[t][r]));
                            ds[t][r] = p[t][r] * dp[t][r];
                        }
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 0 ? !L : !R) continue;
                        sv[t].add(dt, Weights4<T>(p[t]));
                        sk[t].add(qt, Weights4<T>(ds[t]));
                    }
                    if (DBIAS) {   // (outside the window, and NaN: 0)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if (R) Table::add_int(cell + 16 - r * 4, held[r] + Table::to_int(ds[1][r], up));
                            if (!R && bx > 0) Table::add_int(cell + 16 - r * 4, held[r]);
                            held[r] = L ? Table::to_int(ds[0][r], up) : 0;
                        }
                        if (poisoned) {
#pragma unroll
                            for (int t = 0; t < 2; ++t) {
                                if (t == 0 ? !L : !R) continue;
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const int c = (cell - table0 - (g.copies > 1 ? copy_offset(own_lane() >> 4, cells) * Table::kIntBytes : 0)) / 4 + 4 * t - r;
                                    const bool in = rowok && (unsigned)(4 * bx + r - (spans[t] & 0xffff)) < (unsigned)spans[t] >> 16;
                                    if (in && !(fabsf(ds[t][r]) < INFINITY)) __hip_atomic_fetch_or(lds_ptr<unsigned>(flags0 + (c >> 5) * 4), 1u << (c & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                                }
                            }
                        }
                    }
                    if (L) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) before[r] = here[r];
                    }
                    a0 += 4 * POSB;
                    t0 += 4 * POSB;
                    l0 += 16;
                    cell -= 16;
                    brow -= 16;
                };
                int bx = 0;
                for (; bx < r_first; ++bx) block(IntC<1>{}, IntC<0>{}, bx);
                for (; bx <= l_last; ++bx) block(IntC<1>{}, IntC<1>{}, bx);
                for (; bx <= r_last; ++bx) block(IntC<0>{}, IntC<1>{}, bx);
                if (DBIAS && r_last == l_last) {   // the left patch's dS of the last block
#pragma unroll
                    for (int r = 0; r < 4; ++r) Table::add_int(cell + 16 - r * 4, held[r]);
                }
            }
            if (g.nstage == 1 && (!last || b + 1 < work.b_end)) {
                workgroup_sync();   // nobody still reads the rows
                issue(last ? b + 1 : b, last ? 0 : s + 1, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) sk[t].settle(), sv[t].settle();
        if (DBIAS) {
            workgroup_sync();   // every wave has added its part; nobody adds more before the next step's barrier
            for (int i = wave * kWave + own_lane(); i < cells; i += kPatchThreads)
                *lds_ptr<typename Table::Sum>(sums0 + i * Table::kSumBytes) += (typename Table::Sum)take_ints<T>(table0, i, cells, g.copies) * (typename Table::Sum)down;
        }
        if (!active) continue;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int lv = own_lane();
            if (sy0 + ((lv & 15) >> 2) < H && px0 + (lv & 3) + 4 * t < W) {
                const unsigned o = key_offset(lv, 4 * t);
                sk[t].store(reinterpret_cast<char *>(dk) + plane_off, o, lv >> 4, scale);
                sv[t].store(reinterpret_cast<char *>(dv) + plane_off, o, lv >> 4, 1.f);
            }
            const float odd = sk[t].not_finite() + sv[t].not_finite();
            const unsigned long long again = __ballot(odd != odd);
            if (again) keys_once_more<T, D>(again, q, k, v, dout, rpb, scale, ld, dk, dv, plane, head, sy0, px0 + 4 * t, g);
        }
    }
    if (DBIAS) write_bias_sums<T>(partial, sums0, flags0, work, head, cells, wave * kWave + own_lane(), g);
}

// ---- host ------------------------------------------------------------------------------------------------------------
struct PatchPlan {
    PatchShape q, kv;
    int lds_q, lds_kv;
    bool ok, pairs, two;   // part 2: pairs of waves to a patch, or two patches to a wave
};
int query_bytes(const Problem &p) { return 4 * (p.dtype == NA2D_F32 ? kQueryWords<float> : kQueryWords<f16_t>); }
// Pairs of waves in part 2: where one wave per patch leaves half of the chip's 4096 places for waves free, wide windows in 16 bit last as long as
// the patch of a border takes (81 blocks at k = 21, one inside 36).  us of both parts and the bias gradient, fp16, 32 channels, one wave / two: k = 15
// 40 / 34 at 256 patches, 44 / 39 at 1300, 43 / 42 at 2048, 60 / 67 at 4096; k = 21 62 / 48, 64 / 53, 66 / 62, 92 / 95.  Between (16 to 64 channels, three
// maps, two waves' time over one's): k = 15 0.89 .. 1.04 to 2600 patches, 0.93 .. 1.14 from there; k = 21 0.87 .. 1.00 to 2600, 0.91 .. 1.05 from there.
bool pairs_wanted(const Problem &p) {
    return p.dtype != NA2D_F32 && p.K > 13 && p.D <= 64 && (long long)p.planes() * ((p.H + 3) / 4) * ((p.W + 3) / 4) <= 2048;
}
// Two patches to a wave in both parts, in 16 bit with up to 32 channels (64: the registers leave two waves to a SIMD, 123 / 131 us at k = 7), from as many patches on as the chip
// has places for waves, where half as many workgroups, which last 1.5 to 1.7 times as long, end earlier.  The rounds of both grids tell (in fifths, one patch / two): us of both parts and the bias
// gradient, one patch / two, k = 11 and k = 13, 56 x 56 10 / 5 (32 planes) 72 / 65 and 76 / 66, 18 / 10 (62) 116 / 108 and 125 / 110, 35 / 18 (128) 221 / 184 and 241 / 186, 28 x 28 10 / 5 (127) 71 / 63 and 82 / 70, 18 / 10
// (245) 118 / 113 and 134 / 127, k = 15 and 21 15 / 8 (184) 117 / 113 and 172 / 149; left alone 56 x 56 8 / 5 (22) 60 / 65 and 62 / 65, 13 / 8 (42) 86 / 89 and 94 / 90, 28 x 28 8 / 5 (86) 59 / 62 and 67 / 69, 13 / 8 (166)
// 88 / 90 and 101 / 103, 64 x 100, k = 15 and 21, 8 / 5 (11) 83 / 79 and 118 / 124.  With up to 256 workgroups 56 x 56 5 / 3 (18) 43 / 49 and 46 / 49.
// Less is enough where a tile's waves meet the same blocks: on maps at most a pair wider than the window, 14 x 14 8 / 5 (263) 51 / 50 and 56 / 52, 13 x 13 13 / 8 (513) 76 / 71 and 86 / 73, 17 x 17 13 / 8 (224) 74 / 67 and
// 81 / 69, and in tiles of 8 columns over all rows of a low map, 21 x 35 8 / 5 (78) 61 / 54 and 67 / 60, 20 / 13 (223) 128 / 124 and 142 / 132, 18 x 39, k = 13, 13 / 8 (103) 81 / 73, 25 x 34, k = 21, 8 / 5 (66) 115 / 103; 31 x 37, k = 15, 8 / 5 (52) 75 / 82.
bool two_wanted(const Problem &p, int one, const PatchShape &two) {   // one: workgroups per item
    const long long n = (long long)two.units * p.B, r1 = fifths_of_rounds((long long)one * p.B), r2 = fifths_of_rounds(n);
    const bool alike = p.W <= p.K + 8 || (two.lg_cols == 0 && p.H <= 28);
    return n > kPlaces / 2 && (alike ? 2 * r1 >= 3 * r2 : 3 * r1 >= 5 * r2);
}
PatchPlan patch_plan(const Problem &p, bool bias, bool dbias) {
    PatchPlan pl{};
    const int K = p.K, posb = p.D * p.elem_bytes(), pitch = bias_pitch(K), cells = (2 * K - 1) * pitch;
    const int table = bias_rows(K, bias) * pitch * 4;
    const auto sums = [&](int copies) { return !dbias ? 0 : p.dtype == NA2D_F32 ? dbias_bytes<float>(cells, copies) : dbias_bytes<f16_t>(cells, copies); };
    // the tile's shape: the one that takes the fewest steps of four streamed rows
    int lg = 3;
    long long least = LLONG_MAX;
    for (int l = 3; l >= 1; --l) {
        const int rows = (32 >> l) + K - 1 < p.H ? (32 >> l) + K - 1 : p.H;
        const long long steps = (long long)((p.W + (4 << l) - 1) / (4 << l)) * ((p.H + (32 >> l) - 1) / (32 >> l)) * ((rows + 3) / 4);
        if (steps < least) least = steps, lg = l;
    }
    const int tw = 4 << lg, th = 32 >> lg;
    const int tiles_x = (p.W + tw - 1) / tw, tiles_y = (p.H + th - 1) / th;
    const int rwq = image_row(p.W, K, tw, posb, [&](int x) { return win_start(x, p.W, K); }, [&](int x) { return win_start(x, p.W, K) + K - 1; });
    const int rwkv = image_row(p.W, K, tw, posb, [&](int x) { return inv_first(x, p.W, K); }, [&](int x) { return inv_last(x, p.W, K); });
    UnitSplit us;
    us.units = tiles_x * tiles_y * p.heads;
    // more workgroups than fit at a time: those next to the borders have up to twice the work, and what waits fills the gaps
    us.splits = 2048 / us.units;
    us.splits = us.splits < 1 ? 1 : us.splits < p.B ? us.splits : p.B;
    us.gd = make_grid_decode(tiles_x, tiles_y, p.heads, p.B, us.splits);
    PatchShape s{p.H, p.W, K, p.heads, tiles_y, us.units, us.splits, rwq, 0, lg, 0, 1, bias ? 1 : 0, dbias ? 1 : 0, us.gd, make_fastdiv(pitch)};
    pl.q = s;
    s.rw = rwkv;
    pl.kv = s;
    pl.q.nstage = image_buffers(table, 2 * 4 * rwq * posb, pl.lds_q);
    // four copies of the integers where they cost neither a buffer nor the second workgroup
    const int stage = 2 * 4 * rwkv * posb + 4 * rwkv * query_bytes(p);
    int lds4 = 0;
    pl.kv.nstage = image_buffers(table + sums(1), stage, pl.lds_kv);
    pl.kv.copies = 1;
    if (dbias && pl.kv.nstage > 0 && image_buffers(table + sums(4), stage, lds4) == pl.kv.nstage && (lds4 <= 80 * 1024 || pl.lds_kv > 80 * 1024)) {
        pl.kv.copies = 4;
        pl.lds_kv = lds4;
    }
    pl.ok = pl.q.nstage > 0 && pl.kv.nstage > 0;
    const bool wide = p.dtype != NA2D_F32 && p.D <= 32 && (long long)p.planes() * ((p.H + 3) / 4) * ((p.W + 3) / 4) >= 4096;
    if (pl.ok && wide) {
        // Each part: the tile with the least steps whose buffers leave room for a second workgroup.  (What looks at the tables takes both, whatever the call has: the number of
        // partial bias gradients follows from the choice.)
        const int room = 80 * 1024, bias_table = bias_rows(K, true) * pitch * 4;
        const auto shape = [&](int fixed, int record, int most_tiles, auto first, auto last, PatchShape &of) {   // record: bytes per streamed position beside its vectors
            long long fewest = LLONG_MAX;
            for (int l = 2; l >= 0; --l) {
                const int w = 8 << l, h = 32 >> l, rows = h + K - 1 < p.H ? h + K - 1 : p.H;
                const int rw = image_row(p.W, K, w, posb, first, last, 8), step = 4 * rw * (2 * posb + record), tx = (p.W + w - 1) / w, ty = (p.H + h - 1) / h;
                const long long steps2 = (long long)tx * ty * ((rows + 3) / 4);
                if (fixed + step > room || steps2 >= fewest || tx * ty > most_tiles) continue;
                fewest = steps2;
                of = s;
                of.rw = rw;
                of.lg_cols = l;
                of.tiles_y = ty;
                of.units = tx * ty * p.heads;
                // a plane per workgroup, so that a compute unit gets tiles next to borders and others alike, until the partial bias gradients would be many
                of.splits = 8192 / of.units;
                of.splits = of.splits < 1 ? 1 : of.splits < p.B ? of.splits : p.B;
                of.gd = make_grid_decode(tx, ty, p.heads, p.B, of.splits);
                of.nstage = fixed + 2 * step <= room ? 2 : 1;
                of.two = 1;
            }
            return fewest < LLONG_MAX;
        };
        PatchShape q2, kv2;   // (part 2: with more than 5/8 as many tiles as with one patch to a wave too many waves have no pair)
        if (shape(bias_table, 0, INT_MAX, [&](int x) { return win_start(x, p.W, K); }, [&](int x) { return win_start(x, p.W, K) + K - 1; }, q2) &&
            shape(bias_table + dbias_bytes<f16_t>(cells, 1), query_bytes(p), tiles_x * tiles_y * 5 / 8, [&](int x) { return inv_first(x, p.W, K); }, [&](int x) { return inv_last(x, p.W, K); }, kv2) &&
            two_wanted(p, us.units, kv2)) {
            pl.two = true;
            const int step_q = 4 * q2.rw * 2 * posb, step_kv = 4 * kv2.rw * (2 * posb + query_bytes(p));
            q2.nstage = table + 2 * step_q <= room ? 2 : 1;
            kv2.copies = dbias && table + sums(4) + kv2.nstage * step_kv <= room ? 4 : 1;
            pl.q = q2;
            pl.kv = kv2;
            pl.lds_q = table + q2.nstage * step_q;
            pl.lds_kv = table + sums(kv2.copies) + kv2.nstage * step_kv;
        }
    }
    if (pl.ok && pairs_wanted(p)) {
        // (whether there are pairs is decided as with both tables: the number of partial bias gradients follows from it)
        const int most = bias_rows(K, true) * pitch * 4, ints = table_bytes<f16_t>(cells, 1) + flag_bytes(cells), joined = 4 * (p.D / 16) * 2048;
        long long fewest = LLONG_MAX;
        for (int l = 2; l >= 0; --l) {
            const int w = 4 << l, h = 16 >> l, rows = h + K - 1 < p.H ? h + K - 1 : p.H;
            const int rw = image_row(p.W, K, w, posb, [&](int x) { return inv_first(x, p.W, K); }, [&](int x) { return inv_last(x, p.W, K); });
            const int step = 2 * 8 * rw * posb + 8 * rw * query_bytes(p), need = step > joined ? step : joined;
            if (most + ints + need > 80 * 1024) continue;   // two workgroups per compute unit, or the second wave of a patch gains nothing
            const int tx = (p.W + w - 1) / w, ty = (p.H + h - 1) / h;
            const long long steps2 = (long long)tx * ty * ((rows + 7) / 8);
            if (steps2 >= fewest) continue;
            fewest = steps2;
            pl.pairs = true;
            const int fixed = table + (dbias ? ints : 0), fixed4 = table + (dbias ? table_bytes<f16_t>(cells, 4) + flag_bytes(cells) : 0);
            pl.kv = s;
            pl.kv.rw = rw;
            pl.kv.lg_split = 1;
            pl.kv.lg_cols = l;
            pl.kv.tiles_y = ty;
            pl.kv.units = tx * ty * p.heads;
            pl.kv.splits = p.B;
            pl.kv.gd = make_grid_decode(tx, ty, p.heads, p.B, p.B);
            pl.kv.nstage = fixed + 2 * step <= 80 * 1024 ? 2 : 1;
            pl.lds_kv = fixed + (pl.kv.nstage == 2 ? 2 * step : need);
            pl.kv.copies = 1;
            if (dbias && fixed4 - fixed + pl.lds_kv <= 80 * 1024) pl.kv.copies = 4, pl.lds_kv += fixed4 - fixed;
        }
    }
    return pl;
}

size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }
size_t bound_count(const Problem &p) { return (size_t)p.planes() * ((p.H + 3) / 4) * ((p.W + 3) / 4); }

template <typename T, int D>
hipError_t launch_patch_bwd_t(const Problem &p, const PatchPlan &pl, const T *q, const T *k, const T *v, const T *rpb, float scale,
                              const float *lse, const T *dout, T *dq, T *dk, T *dv, float *ld, uint32_t *bound, float *partial, hipStream_t s) {
    const dim3 grid_q(xcd_padded_grid(pl.q.units * pl.q.splits)), grid_kv(xcd_padded_grid(pl.kv.units * pl.kv.splits)), threads(kPatchThreads);
    const auto launch = [&](auto kern, LdsAllowed &allowed, dim3 grid, int lds, auto... args) -> hipError_t {
        if (hipError_t e = allow_lds(kern, 160 * 1024, allowed); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, threads, lds, s, args...);
        return hipGetLastError();
    };
    if constexpr (D <= 32 && sizeof(T) == 2) {
        if (pl.two) {
            static LdsAllowed allowed_q2, allowed_kv2[2];
            if (hipError_t e = launch(patch_bwd_q2_kernel<T, D>, allowed_q2, grid_q, pl.lds_q, q, k, v, rpb, scale, lse, dout, dq, ld, bound, pl.q); e != hipSuccess) return e;
            return launch(partial ? patch_bwd_kv2_kernel<T, D, true> : patch_bwd_kv2_kernel<T, D, false>, allowed_kv2[partial != nullptr], grid_kv, pl.lds_kv, q, k, v, rpb, scale, ld,
                          bound, dout, dk, dv, partial, pl.kv);
        }
    }
    static LdsAllowed allowed_q, allowed_kv, allowed_pairs;
    if (hipError_t e = launch(patch_bwd_q_kernel<T, D>, allowed_q, grid_q, pl.lds_q, q, k, v, rpb, scale, lse, dout, dq, ld, bound, pl.q); e != hipSuccess) return e;
    if constexpr (D * sizeof(T) <= 128 && sizeof(T) == 2) {
        if (pl.pairs) return launch(patch_bwd_kv_kernel<T, D, 1>, allowed_pairs, grid_kv, pl.lds_kv, q, k, v, rpb, scale, ld, bound, dout, dk, dv, partial, pl.kv);
    }
    return launch(patch_bwd_kv_kernel<T, D, 0>, allowed_kv, grid_kv, pl.lds_kv, q, k, v, rpb, scale, ld, bound, dout, dk, dv, partial, pl.kv);
}

}  // namespace

// Where the two kernels are the faster ones, time over that of recomputing the weights into memory and the unfused steps (with the bias
// gradient; 14 x 14, 33 x 70 and 56 x 56 maps; a wave works its patch off alone, so that a call of few tiles lasts as long as one tile).
// 16 bit, to 64 channels: 0.23 .. 0.9, but 64 channels with k >= 15 1.25 .. 1.45 at 27 tiles (0.68 at 135).  128 channels: k <= 11
// 0.9 .. 1.7; k >= 13 1.1 .. 2.4 at up to 135 tiles, 0.63 .. 0.95 at 1000.  fp32, 16 channels: 0.5 .. 0.99, but k >= 11 1.1 .. 1.4 at 8
// and 27 tiles (0.73 .. 0.9 at 84 and more).  fp32, 32 channels: k = 3 0.8 .. 1.08, the large calls above 1; k = 5 0.6 .. 0.95; beyond 1.2 .. 1.9 at
// 27 tiles, 0.82 .. 1.09 at 84, 0.74 .. 1.0 at 135, 0.5 .. 0.85 at 1000.  fp32, 64 channels: k = 3 0.9 .. 1.5; beyond 1.0 .. 2.4 to 135 tiles, and at 1000
// 0.64 .. 0.93, but 0.97 .. 1.27 on maps narrower than a tile of 32.  128 channels in fp32: the registers do not hold a wave's sums.
bool patch_bwd_supported(const Problem &p) {
    if (fused_bwd_supported(p) || p.D * p.elem_bytes() > 256) return false;
    const PatchPlan pl = patch_plan(p, true, true);
    if (!pl.ok) return false;
    const long long tiles = (long long)pl.q.units * p.B;
    if (p.dtype != NA2D_F32) return p.D <= 32 || (p.D == 64 && (p.K <= 13 || tiles >= 64)) || (p.D == 128 && p.K >= 13 && tiles >= 512);
    if (p.D == 16) return p.K <= 9 || tiles >= 64;
    if (p.D == 32) return p.K == 5 || (p.K >= 7 && tiles >= 128);
    return p.K >= 5 && p.W >= 32 && tiles >= 512;
}

// (log2(e) lse, delta) per query, a bound per query patch, a partial bias gradient per workgroup of part 2
size_t patch_bwd_workspace_bytes(const Problem &p) {
    const PatchPlan pl = patch_plan(p, true, true);
    const int nb = 2 * p.K - 1;
    return up256(p.queries() * query_bytes(p)) + up256(bound_count(p) * 4) + up256((size_t)pl.kv.units * pl.kv.splits * rpb_cell_stride(nb * nb) * 4);
}

hipError_t launch_patch_bwd(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, const float *lse,
                            const void *dout, void *dq, void *dk, void *dv, BiasOut d_rpb, void *workspace, hipStream_t s) {
    const PatchPlan pl = patch_plan(p, rpb != nullptr, (bool)d_rpb);
    if (!pl.ok) return hipErrorInvalidValue;
    char *ws = static_cast<char *>(workspace);
    float *ld = reinterpret_cast<float *>(ws);
    uint32_t *bound = d_rpb ? reinterpret_cast<uint32_t *>(ws + up256(p.queries() * query_bytes(p))) : nullptr;
    float *partial = d_rpb ? reinterpret_cast<float *>(ws + up256(p.queries() * query_bytes(p)) + up256(bound_count(p) * 4)) : nullptr;
    hipError_t e = hipErrorInvalidValue;
    const auto run = [&]() -> hipError_t {
        NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, if constexpr (D * sizeof(T) <= 256) return (launch_patch_bwd_t<T, D>(p, pl,
            static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v), static_cast<const T *>(rpb), scale, lse,
            static_cast<const T *>(dout), static_cast<T *>(dq), static_cast<T *>(dk), static_cast<T *>(dv), ld, bound, partial, s))));
        return hipErrorInvalidValue;
    };
    e = run();
    if (e != hipSuccess || !d_rpb) return e;
    return launch_rpb_final_av(p, partial, d_rpb, AvRpbSplit{pl.kv.units / p.heads, pl.kv.splits}, s);
}

}  // namespace na2d
