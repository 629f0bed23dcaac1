// Fused 1D neighbourhood attention backward on the matrix cores, f16 / bf16 (arXiv 2204.07143: Eq. 2-4 differentiated, on a sequence):
// dq, dk, dv and the bias gradient from q, k, v, dout and the forward's log-sum-exp, in groups of 16 positions against blocks of 16 as in the
// fused forward.
//   P[i, j] = exp(scale <q_i, k_j> + B(i, j) - lse_i)   dP[i, j] = <dout_i, v_j>   delta_i = sum_j P dP   dS = P (dP - delta_i)
// Query side: 16 queries, the NBLK = ceil((k + 15) / 16) blocks of keys their windows reach; P and dP stay in registers, so that one sweep gives
// delta and dq_i = scale sum_j dS k_j.  Key side: 16 keys and the queries that see them, NBLK blocks at a time (clear of the ends that is all of
// them): dv_j = sum_i P dout_i, dk_j = scale sum_i dS q_i.
// P and dS enter the sums as two 16-bit halves (22 digits in fp16, 16 in bf16).  In fp16 a column's dS are scaled by the power of two that
// brings the largest near 2^15, so that the result does not depend on the scale of dout.
// Bias gradient: clear of the ends a lane's cells are the same for each of its groups, so that it adds them up in registers, in 64 bits; then they
// join the workgroup's table as 64-bit fixed-point integers (integer additions commute: the result is bitwise reproducible).
// A masked product is 0 * x: results that are not finite are computed once more from their own window.
// Up to k = 17 one kernel does both sides for most calls (below).
// Measured at 64 x 2 x 3136 queries, fp16, the call (a thread per position on the plain ALU before): k = 7 46.9 us (72), in two kernels 24.5 the query side and 29.9 the key
// side at 5.2 TB/s; k = 31 62.4 (163); k = 63 85 (369), where the vector instructions of 5 blocks show.
#include "lds_attr.hpp"
#include "na1d_common.hpp"
#include "na1d_kernels.hpp"

namespace na1d {

using namespace na2d;

namespace {

constexpr int kWaves = 4, kThreads = kWaves * kWave, kGroups = 4;   // groups per wave
constexpr int kTile = kWaves * kGroups * kGroup;
static_assert(kTile == 256, "the partial bias gradients are one per 256 positions");

__host__ __device__ constexpr int up16(int n) { return (n + 15) & ~15; }

// the power of two that brings `most` near 2^15, as an exponent
__device__ __forceinline__ int lift(float most) {
    const int e = 15 - __builtin_amdgcn_frexp_expf(most);
    return e < 100 ? e : 100;   // (2^100 and its inverse are floats)
}

// The four lanes of a column work on it, eight channels each (8 g .. 8 g + 7), which they hold on return.  What it meets lies in LDS.
// (us of the backward at 64 x 2 x 3136, fp16, k = 31, with one infinite key per plane 118, dout all infinite 191, v or dout all NaN 77, finite 62; with the
// vectors read from memory, one position at a time, 191, 361 and 85.  k = 63: 214, 403, 106 and 85.)
template <typename T> struct Pairs {   // kOnceMore positions from `at` on: weights, upstream products, the position's two vectors
    VecN<T, 8> x[kOnceMore], y[kOnceMore];
    float p[kOnceMore], dp[kOnceMore];
};
// p and dp of positions at .. at + kOnceMore - 1 against the lane's own two vectors; xa, ya: the lane's part of position 0 in the two images; bias and
// lse2 of a position
template <typename T, typename Bias, typename Lse>
__device__ __forceinline__ void work_out(Pairs<T> &w, const VecN<T, 8> &own_x, const VecN<T, 8> &own_y, int xa, int ya, int at, int n, float scale2, Bias bias, Lse lse2) {
#pragma unroll
    for (int e = 0; e < kOnceMore; ++e) {
        const int pos = at + e < n ? at + e : n - 1;   // (past the end: once more, not added)
        load8_lds(w.x[e], xa + pos * kBytes);
        load8_lds(w.y[e], ya + pos * kBytes);
        w.p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, group_sum(dot32(own_x, w.x[e])), bias(pos)) - lse2(pos));
        w.dp[e] = group_sum(dot32(own_y, w.y[e]));
    }
}
template <typename F> __device__ __forceinline__ void add_cell(int table, int cell, F ds) {
    __hip_atomic_fetch_add(lds_ptr<unsigned long long>(table + cell * 8), (unsigned long long)to_fixed42(ds), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One query from its own window: delta, channels 8 g .. 8 g + 7 of dq, and (lane group 0) its part of the bias gradient.  own: its q and dout;
// ka, va: the lane's part of the window's first key and value; bias: of the window's first slot; cell: its cell's number.
template <typename T>
__device__ void query_once_more(const VecN<T, 8> (&own)[2], int ka, int va, const float *bias, float scale, int K, int g, float lse2, int table, int cell, float (&x)[8],
                                float &delta) {
    const float scale2 = scale * kLog2e;
    const auto bias_of = [&](int a) { return bias[a]; };
    const auto lse_of = [&](int) { return lse2; };
    delta = 0.f;
#pragma unroll 1
    for (int a = 0; a < K && delta == delta; a += kOnceMore) {
        Pairs<T> w;
        work_out(w, own[0], own[1], ka, va, a, K, scale2, bias_of, lse_of);
#pragma unroll
        for (int e = 0; e < kOnceMore; ++e) delta = a + e < K ? __builtin_fmaf(w.p[e], w.dp[e], delta) : delta;
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) x[d] = delta == delta ? 0.f : NAN;   // (every dS is NaN then, and counts as 0 in the bias gradient)
#pragma unroll 1
    for (int a = 0; a < K && delta == delta; a += kOnceMore) {
        Pairs<T> w;
        work_out(w, own[0], own[1], ka, va, a, K, scale2, bias_of, lse_of);
#pragma unroll
        for (int e = 0; e < kOnceMore; ++e)
            if (a + e < K) {
                const float ds = w.p[e] * (w.dp[e] - delta);
                axpy32(x, ds, w.x[e]);
                if (table && g == 0) add_cell(table, cell + a + e, ds);
            }
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) x[d] *= scale;
}
// One key from the n queries that see it, likewise; a gradient that is finite in all four lanes stays.  own: its k and v; qa, da: the lane's part of
// the first query and its upstream gradient; ld: that query's (lse, delta); bias: of the first query's cell (those that follow lie in front of it).
template <typename T>
__device__ void key_once_more(const VecN<T, 8> (&own)[2], int qa, int da, int ld, const float *bias, float scale, int n, float (&xk)[8], float (&xv)[8]) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const float scale2 = scale * kLog2e;
    float ak[8], av[8], nk = 0.f, nv = 0.f;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        nk = __builtin_fmaf(xk[d], 0.f, nk);
        nv = __builtin_fmaf(xv[d], 0.f, nv);
        ak[d] = av[d] = 0.f;
    }
    const bool want_k = group_sum(nk) != 0.f, want_v = group_sum(nv) != 0.f;   // (0 or NaN)
#pragma unroll 1
    for (int a = 0; a < n; a += kOnceMore) {
        Pairs<T> w;
        work_out(w, own[0], own[1], qa, da, a, n, scale2, [&](int u) { return bias[-u]; }, [&](int u) { return (*lds_ptr<f32x2_t>(ld + u * 8)).x; });
#pragma unroll
        for (int e = 0; e < kOnceMore; ++e)
            if (a + e < n) {
                axpy32(av, w.p[e], w.y[e]);
                axpy32(ak, w.p[e] * (w.dp[e] - (*lds_ptr<f32x2_t>(ld + (a + e) * 8)).y), w.x[e]);
            }
        float open = 0.f;   // (what is NaN stays NaN: not 0 while some wanted sum is still a number)
#pragma unroll
        for (int d = 0; d < 8; ++d) open = (want_k && ak[d] == ak[d]) || (want_v && av[d] == av[d]) ? 1.f : open;
        if (group_sum(open) == 0.f) break;
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        if (want_k) xk[d] = ak[d] * scale;
        if (want_v) xv[d] = av[d];
    }
}

template <int NBLK> constexpr int kQueryRows = kTile - kGroup + 16 * NBLK;   // keys staged
// both images, the bias as each lane of a group clear of the ends meets it, the bias and the integers of its gradient
__host__ __device__ constexpr int query_lds(int nblk, int K) {
    return 2 * (kTile - kGroup + 16 * nblk) * kBytes + nblk * kWave * 16 + up16((2 * K - 1) * 4) + (2 * K - 1) * 8;
}

template <typename T, int NBLK>
__global__ __launch_bounds__(kThreads, (NBLK > 3 ? 3 : 4)) void bwd1d_q_mfma_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale, const float *__restrict__ lse,
    const T *__restrict__ dout, T *__restrict__ dq, float *__restrict__ delta_out, long long *__restrict__ partial, int L, int heads, int K, int tiles) {
    constexpr int kImage = kQueryRows<NBLK> * kBytes;
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave), j = lane & 15, g = lane >> 4;
    const int plane = blockIdx.x / tiles, t0 = (blockIdx.x - plane * tiles) * kTile, NB = 2 * K - 1, R = K >> 1;
    const size_t first = (size_t)plane * L;
    constexpr int kInner = NBLK * kWave * 16;
    const int h0 = win_start(t0, L, K), img = lds_addr(lds), inner = img + 2 * kImage, cells = inner + kInner + up16(NB * 4), table = partial ? cells : 0;
    float *bias = reinterpret_cast<float *>(lds + 2 * kImage + kInner);
    stage_pair<kWaves>(reinterpret_cast<const char *>(k) + (first + h0) * kBytes, reinterpret_cast<const char *>(v) + (first + h0) * kBytes, L - 1 - h0,
                       kQueryRows<NBLK>, img, img + kImage, wave, lane);
    const T *own_rpb = rpb ? rpb + (size_t)(plane % heads) * NB : nullptr;
    for (int u = tid; u < NB; u += kThreads) {
        bias[u] = own_rpb ? to_f32(own_rpb[u]) * kLog2e : 0.f;
        if (partial) *lds_ptr<unsigned long long>(cells + u * 8) = 0ull;
    }
#pragma unroll
    for (int u = tid; u < NBLK * kWave * 4; u += kThreads) {   // (block, lane, result)
        const int a = 16 * (u >> 8) + 4 * ((u >> 6) & 3) + (u & 3) - ((u >> 2) & 15);   // slot in the window
        const bool in = (unsigned)a < (unsigned)K;
        const float t = own_rpb && in ? to_f32(own_rpb[a + K - 1 - R]) * kLog2e : 0.f;
        *lds_ptr<float>(inner + u * 4) = in ? t : -INFINITY;
    }
    u32x4 qv, gv;
    float lse_i;
    auto load = [&](int n) {
        const int i = t0 + (wave * kGroups + n) * kGroup + j;
        const size_t at = first + (i < L ? i : L - 1);
        qv = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(q) + at * kBytes + g * 16);
        gv = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(dout) + at * kBytes + g * 16);
        lse_i = lse[at];
    };
    load(0);
    wait_global_loads();
    workgroup_sync();

    const float scale2 = scale * kLog2e;
    double sums[NBLK][4];   // (four fp32 numbers to 2^-42 and beyond)
#pragma unroll
    for (int c = 0; c < NBLK; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[c][r] = 0.;
#pragma unroll 1
    for (int n = 0; n < kGroups; ++n) {
        const int i0 = t0 + (wave * kGroups + n) * kGroup;
        if (i0 >= L) break;
        const int o = win_start(i0, L, K), i = i0 + j < L ? i0 + j : L - 1;
        const int w = win_start(i, L, K) - o;   // the lane's window begins at position w of the blocks
        const bool clear = o == i0 - R && i0 + kGroup - 1 + R < L;
        f32x4 b[NBLK];
        if (clear) {
#pragma unroll
            for (int c = 0; c < NBLK; ++c) b[c] = *lds_ptr<f32x4>(inner + c * (kWave * 16) + lane * 16);
        } else {
#pragma unroll
            for (int c = 0; c < NBLK; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = 16 * c + 4 * g + r;
                    const bool in = (unsigned)(at - w) < (unsigned)K;
                    const float t = bias[in ? at + o - i + K - 1 : 0];
                    b[c][r] = in ? t : -INFINITY;
                }
        }
        const int ka = row_addr(img, o - h0, j, g);
        const float lse2 = lse_i * kLog2e;
        f32x4 s[NBLK], dp[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) {
            s[c] = mfma_16x16x32<T>(*lds_ptr<u32x4>(ka + c * kGroup * kBytes), qv, f32x4{0.f, 0.f, 0.f, 0.f});
            dp[c] = mfma_16x16x32<T>(*lds_ptr<u32x4>(ka + kImage + c * kGroup * kBytes), gv, f32x4{0.f, 0.f, 0.f, 0.f});
        }
        if (NBLK != 3 && n + 1 < kGroups) load(n + 1);
        float delta = 0.f;
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s[c][r], b[c][r]) - lse2);
                delta = __builtin_fmaf(s[c][r], dp[c][r], delta);
            }
        delta = group_sum(delta);
        float most = 0.f;
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] *= dp[c][r] - delta;
                most = fmaxf(most, fabsf(s[c][r]));
            }
        const int e = kShift<T> != 0.f ? lift(group_max(most)) : 0;
        const float up = __builtin_ldexpf(1.f, e);
        Split4<T> ws[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) {
            const float t[4] = {s[c][0] * up, s[c][1] * up, s[c][2] * up, s[c][3] * up};
            ws[c].set(t);
        }
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        if (NBLK == 3 && n + 1 < kGroups) load(n + 1);   // (later, for the registers)
        weighted_sum<T, NBLK>(vector_addr(img, o - h0, j, g), ws, acc);
        const float back = scale * __builtin_ldexpf(1.f, -e);
        float x[8], odd = delta * 0.f;   // odd: NaN where something is not finite
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            x[d] = acc[d >> 2][d & 3] * back;
            odd = __builtin_fmaf(x[d], 0.f, odd);
        }
        const unsigned again = marked_columns(odd != odd);
        const bool redo = (again >> j) & 1u, live = i0 + j < L;
        if (partial) {
            if (clear && again == 0 && __ballot(most >= 524288.f) == 0) {   // (2^19: the sum of four stays in the integers' range)
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sums[c][r] += s[c][r];
            } else {
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = 16 * c + 4 * g + r;
                        if (live && !redo && (unsigned)(at - w) < (unsigned)K) add_cell(cells, at + o - i + K - 1, s[c][r]);
                    }
            }
        }
        if (redo && live) {
            VecN<T, 8> own[2];
            load_vec32(own[0], q + (first + i) * kHeadDim + 8 * g);
            load_vec32(own[1], dout + (first + i) * kHeadDim + 8 * g);
            const int s0 = win_start(i, L, K), at = img + (s0 - h0) * kBytes + g * 16, cell = s0 - i + K - 1;
            query_once_more<T>(own, at, at + kImage, bias + cell, scale, K, g, lse2, table, cell, x, delta);
        }
        if (live) {
            store_vector<T>(reinterpret_cast<char *>(dq) + (first + i) * kBytes + g * 16, x);
            if (g == 0) delta_out[first + i] = delta;
        }
    }
    if (partial == nullptr) return;
#pragma unroll
    for (int c = 0; c < NBLK; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = 16 * c + 4 * g + r - j;   // slot in the window
            if ((unsigned)a < (unsigned)K) add_cell(cells, a + K - 1 - R, sums[c][r]);
        }
    workgroup_sync();
    for (int u = tid; u < NB; u += kThreads) partial[(size_t)blockIdx.x * NB + u] = (long long)*lds_ptr<unsigned long long>(cells + u * 8);
}

// The queries that see a tile are at most kTile + 2 (K - 1), and a group's blocks run on by less than NBLK blocks.
__host__ __device__ constexpr int key_rows(int nblk, int K) { return up16(kTile + 2 * (K - 1)) + 16 * nblk; }
__host__ __device__ constexpr int key_lds(int nblk, int K) { return key_rows(nblk, K) * (2 * kBytes + 8) + (2 * K - 1) * 4; }

template <typename T, int NBLK>
__global__ __launch_bounds__(kThreads, (NBLK > 3 ? 3 : 4)) void bwd1d_kv_mfma_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale, const float *__restrict__ lse,
    const float *__restrict__ delta, const T *__restrict__ dout, T *__restrict__ dk, T *__restrict__ dv, int L, int heads, int K, int tiles, RpbTables tables,
    int own_blocks) {
    // (workgroups from own_blocks on add up the bias gradient's tables)
    extern __shared__ __align__(16) char lds[];
    if ((int)blockIdx.x >= own_blocks) {
        static_assert(kThreads == kFinalThreads, "last sum");
        rpb_final_cell(tables, blockIdx.x - own_blocks, lds_addr(lds));
        return;
    }
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave), j = lane & 15, g = lane >> 4;
    const int plane = blockIdx.x / tiles, t0 = (blockIdx.x - plane * tiles) * kTile, t1 = t0 + kTile - 1 < L - 1 ? t0 + kTile - 1 : L - 1, NB = 2 * K - 1;
    const size_t first = (size_t)plane * L;
    const int rows = key_rows(NBLK, K), image = rows * kBytes, img = lds_addr(lds), ld0 = img + 2 * image;
    const int h0 = inv_first(t0, L, K), used = up16(inv_last(t1, L, K) - h0 + 1) + 16 * NBLK;   // (at most `rows`)
    float *bias = reinterpret_cast<float *>(lds + 2 * image + rows * 8);
    stage_pair<kWaves>(reinterpret_cast<const char *>(q) + (first + h0) * kBytes, reinterpret_cast<const char *>(dout) + (first + h0) * kBytes, L - 1 - h0,
                       used, img, img + image, wave, lane);
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    for (int u = tid; u < used; u += kThreads) {   // log2(e) lse and delta of every query
        const size_t at = first + (h0 + u < L - 1 ? h0 + u : L - 1);
        *lds_ptr<f32x2_t>(ld0 + u * 8) = f32x2_t{lse[at] * kLog2e, delta[at]};
    }
    const T *own_rpb = rpb ? rpb + (size_t)(plane % heads) * NB : nullptr;
    for (int u = tid; u < NB; u += kThreads) bias[u] = own_rpb ? to_f32(own_rpb[u]) * kLog2e : 0.f;
    u32x4 kv, vv;
    auto load = [&](int n) {
        const int key = t0 + (wave * kGroups + n) * kGroup + j;
        const size_t at = (first + (key < L ? key : L - 1)) * kBytes + g * 16;
        kv = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(k) + at);
        vv = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(v) + at);
    };
    load(0);
    wait_global_loads();
    workgroup_sync();

    const float scale2 = scale * kLog2e;
    float b[NBLK][4];
    bool inner = false;   // b[] is that of a group clear of the ends
#pragma unroll 1
    for (int n = 0; n < kGroups; ++n) {
        const int j0 = t0 + (wave * kGroups + n) * kGroup;
        if (j0 >= L) break;
        const int j1 = j0 + kGroup - 1 < L - 1 ? j0 + kGroup - 1 : L - 1, key = j0 + j < L ? j0 + j : L - 1;
        const int o = inv_first(j0, L, K), blocks = (inv_last(j1, L, K) - o + kGroup) / kGroup;
        const int lo = inv_first(key, L, K) - o, count = inv_last(key, L, K) - o - lo + 1;   // the queries that see the lane's key
        const bool clear = j0 >= K && j0 + kGroup - 1 < L - K;
        f32x4 ak[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}, av[2] = {ak[0], ak[0]};
        int e = 100;   // ak counts 2^-e
#pragma unroll 1
        for (int c0 = 0; c0 < blocks; c0 += NBLK) {
            if (!(clear && inner)) {
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = 16 * (c0 + c) + 4 * g + r;
                        const bool in = (unsigned)(at - lo) < (unsigned)count;
                        const float t = bias[in ? key - o - at + K - 1 : 0];
                        b[c][r] = in ? t + kShift<T> : -INFINITY;
                    }
                inner = clear;
            }
            const int pos = o - h0 + 16 * c0, qa = row_addr(img, pos, j, g), la = ld0 + (pos + 4 * g) * 8;
            Split4<T> wp[NBLK], ws[NBLK];
            f32x4 ds[NBLK];
            float most = 0.f;
#pragma unroll
            for (int c = 0; c < NBLK; ++c) {
                const f32x4 s = mfma_16x16x32<T>(*lds_ptr<u32x4>(qa + c * kGroup * kBytes), kv, f32x4{0.f, 0.f, 0.f, 0.f});
                const f32x4 dp = mfma_16x16x32<T>(*lds_ptr<u32x4>(qa + image + c * kGroup * kBytes), vv, f32x4{0.f, 0.f, 0.f, 0.f});
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const f32x2_t of = *lds_ptr<f32x2_t>(la + (16 * c + r) * 8);
                    p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s[r], b[c][r]) - of.x);
                    ds[c][r] = p[r] * (dp[r] - of.y);
                    most = fmaxf(most, fabsf(ds[c][r]));
                }
                wp[c].set(p);
            }
            if constexpr (kShift<T> != 0.f) {
                const int lifted = lift(group_max(most)), both = lifted < e ? lifted : e;
                if (c0 > 0) {
                    const float down = __builtin_ldexpf(1.f, both - e);
                    ak[0] *= down;
                    ak[1] *= down;
                }
                e = both;
            } else {
                e = 0;
            }
            const float up = __builtin_ldexpf(1.f, e);
#pragma unroll
            for (int c = 0; c < NBLK; ++c) {
                const float t[4] = {ds[c][0] * up, ds[c][1] * up, ds[c][2] * up, ds[c][3] * up};
                ws[c].set(t);
            }
            weighted_sum<T, NBLK>(vector_addr(img + image, pos, j, g), wp, av);
            weighted_sum<T, NBLK>(vector_addr(img, pos, j, g), ws, ak);
        }
        settle_products<2>(ak);
        settle_products<2>(av);
        if (n + 1 < kGroups) load(n + 1);
        const float back_v = __builtin_ldexpf(1.f, (int)-kShift<T>), back_k = scale * __builtin_ldexpf(1.f, -e - (int)kShift<T>);
        float xk[8], xv[8], odd = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            xk[d] = ak[d >> 2][d & 3] * back_k;
            xv[d] = av[d >> 2][d & 3] * back_v;
            odd = __builtin_fmaf(xk[d], 0.f, __builtin_fmaf(xv[d], 0.f, odd));
        }
        const unsigned again = marked_columns(odd != odd);
        if (j0 + j >= L) continue;
        if ((again >> j) & 1u) {
            VecN<T, 8> own[2];
            load_vec32(own[0], k + (first + key) * kHeadDim + 8 * g);
            load_vec32(own[1], v + (first + key) * kHeadDim + 8 * g);
            const int i0 = inv_first(key, L, K), at = img + (i0 - h0) * kBytes + g * 16;
            key_once_more<T>(own, at, at + image, ld0 + (i0 - h0) * 8, bias + (key - i0 + K - 1), scale, inv_last(key, L, K) - i0 + 1, xk, xv);
        }
        store_vector<T>(reinterpret_cast<char *>(dk) + (first + key) * kBytes + g * 16, xk);
        store_vector<T>(reinterpret_cast<char *>(dv) + (first + key) * kBytes + g * 16, xv);
    }
}

template <typename T, int NBLK>
hipError_t launch_t(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, const float *lse, const void *dout,
                    void *dq, void *dk, void *dv, float *delta, long long *partial, BiasOut d_rpb, hipStream_t s) {
    auto kern_q = bwd1d_q_mfma_kernel<T, NBLK>;
    auto kern_kv = bwd1d_kv_mfma_kernel<T, NBLK>;
    static LdsAllowed allowed_q, allowed_kv;
    if (hipError_t e = allow_lds(kern_q, query_lds(NBLK, kMaxK), allowed_q); e != hipSuccess) return e;
    if (hipError_t e = allow_lds(kern_kv, key_lds(NBLK, kMaxK), allowed_kv); e != hipSuccess) return e;
    const int tiles = (p.L + kTile - 1) / kTile;
    const T *tq = static_cast<const T *>(q), *tk = static_cast<const T *>(k), *tv = static_cast<const T *>(v), *tr = static_cast<const T *>(rpb), *td = static_cast<const T *>(dout);
    hipLaunchKernelGGL(kern_q, dim3(p.planes() * tiles), dim3(kThreads), query_lds(NBLK, p.K), s, tq, tk, tv, tr, scale, lse, td, static_cast<T *>(dq), delta, partial,
                       p.L, p.heads, p.K, tiles);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    const int own_blocks = p.planes() * tiles, NB = 2 * p.K - 1, last_sum = d_rpb ? p.heads * NB : 0;
    const RpbTables tables{partial, d_rpb, p.B, p.heads, tiles, NB};
    const bool along = launch_holds((long long)own_blocks + last_sum, kThreads);
    hipLaunchKernelGGL(kern_kv, dim3(own_blocks + (along ? last_sum : 0)), dim3(kThreads), key_lds(NBLK, p.K), s, tq, tk, tv, tr, scale, lse, delta, td, static_cast<T *>(dk),
                       static_cast<T *>(dv), p.L, p.heads, p.K, tiles, tables, own_blocks);
    if (hipError_t e = hipGetLastError(); e != hipSuccess || along) return e;
    return launch_rpb_final(tables, s);
}

// ---- both sides in one kernel (k <= 17) ---------------------------------------------------------------------------------------
// A workgroup stages a tile of kWholeTile positions with the 16 in front of it and the 16 behind it once for both sides: every query that sees a key of
// the tile (R in front, up to k - 1 behind) and the windows of those queries.  The two kernels are at the memory's rate and read q, k, v and dout once
// each; here that is once in all (with a seventh more for the neighbours, from the L2).  The neighbours' queries are worked out as far as their
// delta.  Groups lie where the two kernels have them, so the results are the same but for the order of the bias gradient's sums.
// Measured (us, the call, two kernels / one): 64 x 2 x 3136 fp16, k = 7 58.2 / 46.9 (44 and the bias gradient's last sum, a launch of its own again; 180 MB at 4.1 TB/s),
// bf16, k = 17 57.2 / 46.2; 256 x 16 x 197 fp16, k = 7 99.7 / 86.4; 1 x 1 x 64 23 / 20.  Wider windows have more neighbours, and their images leave no room for a second
// workgroup on a compute unit.
constexpr int kWholeWaves = 8, kWholeThreads = kWholeWaves * kWave, kWholeGroups = 2, kWholeTile = 14 * kGroup, kWholeK = 17;
static_assert(kWholeWaves * kWholeGroups * kGroup == kWholeTile + 2 * kGroup, "queries of a tile");
constexpr int kWholeKeyRows = kWholeTile + 2 * kGroup - kGroup + 32, kWholeQueryRows = kWholeTile + 2 * kGroup + 32;
// the images, (lse, delta) per query, the bias as each lane of a group clear of the ends meets it, the bias and the integers of its gradient
__host__ __device__ constexpr int whole_lds(int K) {
    return 2 * (kWholeKeyRows + kWholeQueryRows) * kBytes + kWholeQueryRows * 8 + 2 * kWave * 16 + up16((2 * K - 1) * 4) + (2 * K - 1) * 8;
}
static_assert(whole_lds(kWholeK) <= 80 * 1024, "two workgroups share a compute unit");

template <typename T>
__global__ __launch_bounds__(kWholeThreads, 4) void bwd1d_whole_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale, const float *__restrict__ lse,
    const T *__restrict__ dout, T *__restrict__ dq, T *__restrict__ dk, T *__restrict__ dv, long long *__restrict__ partial, int L, int heads, int K, int tiles) {
    constexpr int NBLK = 2, kKeyImage = kWholeKeyRows * kBytes, kQueryImage = kWholeQueryRows * kBytes;
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave), j = lane & 15, g = lane >> 4;
    const int plane = blockIdx.x / tiles, t0 = (blockIdx.x - plane * tiles) * kWholeTile, t1 = t0 + kWholeTile - 1 < L - 1 ? t0 + kWholeTile - 1 : L - 1;
    const int NB = 2 * K - 1, R = K >> 1;
    const size_t first = (size_t)plane * L;
    // the first staged query and key
    const int h0q = t0 - kGroup > 0 ? t0 - kGroup : 0, h0k = win_start(h0q, L, K);
    constexpr int kInner = NBLK * kWave * 16, kLd = 2 * (kKeyImage + kQueryImage), kBias = kLd + kWholeQueryRows * 8 + kInner;
    const int img_k = lds_addr(lds), img_q = img_k + 2 * kKeyImage, ld0 = img_k + kLd, inner = ld0 + kWholeQueryRows * 8, cells = img_k + kBias + up16(NB * 4),
              table = partial ? cells : 0;
    float *bias = reinterpret_cast<float *>(lds + kBias);
    stage_pair<kWholeWaves>(reinterpret_cast<const char *>(k) + (first + h0k) * kBytes, reinterpret_cast<const char *>(v) + (first + h0k) * kBytes, L - 1 - h0k,
                            kWholeKeyRows, img_k, img_k + kKeyImage, wave, lane);
    stage_pair<kWholeWaves>(reinterpret_cast<const char *>(q) + (first + h0q) * kBytes, reinterpret_cast<const char *>(dout) + (first + h0q) * kBytes, L - 1 - h0q,
                            kWholeQueryRows, img_q, img_q + kQueryImage, wave, lane);
    const T *own_rpb = rpb ? rpb + (size_t)(plane % heads) * NB : nullptr;
    for (int u = tid; u < NB; u += kWholeThreads) {
        bias[u] = own_rpb ? to_f32(own_rpb[u]) * kLog2e : 0.f;
        if (partial) *lds_ptr<unsigned long long>(cells + u * 8) = 0ull;
    }
    for (int u = tid; u < kWholeQueryRows; u += kWholeThreads) *lds_ptr<f32x2_t>(ld0 + u * 8) = f32x2_t{0.f, 0.f};   // (rows without a query meet zero weights)
    {
        const int u = tid;   // (block, lane, result)
        static_assert(NBLK * kWave * 4 == kWholeThreads, "entries");
        const int a = 16 * (u >> 8) + 4 * ((u >> 6) & 3) + (u & 3) - ((u >> 2) & 15);   // slot in the window
        const bool in = (unsigned)a < (unsigned)K;
        const float t = own_rpb && in ? to_f32(own_rpb[a + K - 1 - R]) * kLog2e : 0.f;
        *lds_ptr<float>(inner + u * 4) = in ? t : -INFINITY;
    }
    // this wave's two groups of queries, from the one in front of the tile on
    const int g0 = t0 - kGroup + wave * kWholeGroups * kGroup;
    const auto lse_of = [&](int i) { return lse[first + (i < 0 ? 0 : i < L ? i : L - 1)]; };
    float lse0 = lse_of(g0 + j), lse1 = lse_of(g0 + kGroup + j);
    asm volatile("" : "+v"(lse0), "+v"(lse1));   // (their wait goes here)
    wait_global_loads();
    workgroup_sync();

    const float scale2 = scale * kLog2e;
    double sums[NBLK][4];   // (four fp32 numbers to 2^-42 and beyond)
#pragma unroll
    for (int c = 0; c < NBLK; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[c][r] = 0.;
#pragma unroll 1
    for (int n = 0; n < kWholeGroups; ++n) {
        const int i0 = g0 + n * kGroup;
        if (i0 < 0 || i0 >= L) continue;
        const int o = win_start(i0, L, K), i = i0 + j < L ? i0 + j : L - 1;
        const int w = win_start(i, L, K) - o;   // the lane's window begins at position w of the blocks
        const bool clear = o == i0 - R && i0 + kGroup - 1 + R < L;
        f32x4 b[NBLK];
        if (clear) {
#pragma unroll
            for (int c = 0; c < NBLK; ++c) b[c] = *lds_ptr<f32x4>(inner + c * (kWave * 16) + lane * 16);
        } else {
#pragma unroll
            for (int c = 0; c < NBLK; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = 16 * c + 4 * g + r;
                    const bool in = (unsigned)(at - w) < (unsigned)K;
                    const float t = bias[in ? at + o - i + K - 1 : 0];
                    b[c][r] = in ? t : -INFINITY;
                }
        }
        const int ka = row_addr(img_k, o - h0k, j, g), at_q = row_addr(img_q, i0 - h0q, j, g);
        const u32x4 qv = *lds_ptr<u32x4>(at_q), gv = *lds_ptr<u32x4>(at_q + kQueryImage);
        const float lse2 = (n == 0 ? lse0 : lse1) * kLog2e;
        f32x4 s[NBLK], dp[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) {
            s[c] = mfma_16x16x32<T>(*lds_ptr<u32x4>(ka + c * kGroup * kBytes), qv, f32x4{0.f, 0.f, 0.f, 0.f});
            dp[c] = mfma_16x16x32<T>(*lds_ptr<u32x4>(ka + kKeyImage + c * kGroup * kBytes), gv, f32x4{0.f, 0.f, 0.f, 0.f});
        }
        float delta = 0.f;
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s[c][r], b[c][r]) - lse2);
                delta = __builtin_fmaf(s[c][r], dp[c][r], delta);
            }
        delta = group_sum(delta);
        if (i0 < t0 || i0 > t1) {   // the neighbours' queries: their delta is all that is needed
            const unsigned again = marked_columns(delta * 0.f != 0.f);
            if (((again >> j) & 1u) && i0 + j < L) {
                VecN<T, 8> own[2];
                float x[8];
                load_vec32(own[0], q + (first + i) * kHeadDim + 8 * g);
                load_vec32(own[1], dout + (first + i) * kHeadDim + 8 * g);
                const int s0 = win_start(i, L, K), at = img_k + (s0 - h0k) * kBytes + g * 16, cell = s0 - i + K - 1;
                query_once_more<T>(own, at, at + kKeyImage, bias + cell, scale, K, g, lse2, 0, cell, x, delta);
            }
            if (g == 0 && i0 + j < L) *lds_ptr<f32x2_t>(ld0 + (i - h0q) * 8) = f32x2_t{lse2, delta};
            continue;
        }
        float most = 0.f;
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] *= dp[c][r] - delta;
                most = fmaxf(most, fabsf(s[c][r]));
            }
        const int e = kShift<T> != 0.f ? lift(group_max(most)) : 0;
        const float up = __builtin_ldexpf(1.f, e);
        Split4<T> ws[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) {
            const float t[4] = {s[c][0] * up, s[c][1] * up, s[c][2] * up, s[c][3] * up};
            ws[c].set(t);
        }
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        weighted_sum<T, NBLK>(vector_addr(img_k, o - h0k, j, g), ws, acc);
        const float back = scale * __builtin_ldexpf(1.f, -e);
        float x[8], odd = delta * 0.f;   // odd: NaN where something is not finite
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            x[d] = acc[d >> 2][d & 3] * back;
            odd = __builtin_fmaf(x[d], 0.f, odd);
        }
        const unsigned again = marked_columns(odd != odd);
        const bool redo = (again >> j) & 1u, live = i0 + j < L;
        if (partial) {
            if (clear && again == 0 && __ballot(most >= 524288.f) == 0) {   // (2^19: the sum of two stays in the integers' range)
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sums[c][r] += s[c][r];
            } else {
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = 16 * c + 4 * g + r;
                        if (live && !redo && (unsigned)(at - w) < (unsigned)K) add_cell(cells, at + o - i + K - 1, s[c][r]);
                    }
            }
        }
        if (redo && live) {
            VecN<T, 8> own[2];
            load_vec32(own[0], q + (first + i) * kHeadDim + 8 * g);
            load_vec32(own[1], dout + (first + i) * kHeadDim + 8 * g);
            const int s0 = win_start(i, L, K), at = img_k + (s0 - h0k) * kBytes + g * 16, cell = s0 - i + K - 1;
            query_once_more<T>(own, at, at + kKeyImage, bias + cell, scale, K, g, lse2, table, cell, x, delta);
        }
        if (live) {
            store_vector<T>(reinterpret_cast<char *>(dq) + (first + i) * kBytes + g * 16, x);
            if (g == 0) *lds_ptr<f32x2_t>(ld0 + (i - h0q) * 8) = f32x2_t{lse2, delta};
        }
    }
    if (partial) {
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int a = 16 * c + 4 * g + r - j;   // slot in the window
                if ((unsigned)a < (unsigned)K) add_cell(cells, a + K - 1 - R, sums[c][r]);
            }
    }
    workgroup_sync();   // every query's delta and part of the bias gradient
    if (partial)
        for (int u = tid; u < NB; u += kWholeThreads) partial[(size_t)blockIdx.x * NB + u] = (long long)*lds_ptr<unsigned long long>(cells + u * 8);

    float b[NBLK][4];
    bool kept = false;   // b[] is that of a group clear of the ends
#pragma unroll 1
    for (int n = 0; n < kWholeGroups; ++n) {
        const int j0 = t0 + (wave * kWholeGroups + n) * kGroup;
        if (j0 > t1) break;
        const int j1 = j0 + kGroup - 1 < L - 1 ? j0 + kGroup - 1 : L - 1, key = j0 + j < L ? j0 + j : L - 1;
        const int o = inv_first(j0, L, K), blocks = (inv_last(j1, L, K) - o + kGroup) / kGroup;
        const int lo = inv_first(key, L, K) - o, count = inv_last(key, L, K) - o - lo + 1;   // the queries that see the lane's key
        const bool clear = j0 >= K && j0 + kGroup - 1 < L - K;
        const int at_k = row_addr(img_k, (j0 - h0k), 0, g) + (key - j0) * kBytes;
        const u32x4 kv = *lds_ptr<u32x4>(at_k), vv = *lds_ptr<u32x4>(at_k + kKeyImage);
        f32x4 ak[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}, av[2] = {ak[0], ak[0]};
        int e = 100;   // ak counts 2^-e
#pragma unroll 1
        for (int c0 = 0; c0 < blocks; c0 += NBLK) {
            if (!(clear && kept)) {
#pragma unroll
                for (int c = 0; c < NBLK; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = 16 * (c0 + c) + 4 * g + r;
                        const bool in = (unsigned)(at - lo) < (unsigned)count;
                        const float t = bias[in ? key - o - at + K - 1 : 0];
                        b[c][r] = in ? t + kShift<T> : -INFINITY;
                    }
                kept = clear;
            }
            const int pos = o - h0q + 16 * c0, qa = row_addr(img_q, pos, j, g), la = ld0 + (pos + 4 * g) * 8;
            Split4<T> wp[NBLK], ws[NBLK];
            f32x4 ds[NBLK];
            float most = 0.f;
#pragma unroll
            for (int c = 0; c < NBLK; ++c) {
                const f32x4 s = mfma_16x16x32<T>(*lds_ptr<u32x4>(qa + c * kGroup * kBytes), kv, f32x4{0.f, 0.f, 0.f, 0.f});
                const f32x4 dp = mfma_16x16x32<T>(*lds_ptr<u32x4>(qa + kQueryImage + c * kGroup * kBytes), vv, f32x4{0.f, 0.f, 0.f, 0.f});
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const f32x2_t of = *lds_ptr<f32x2_t>(la + (16 * c + r) * 8);
                    p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(scale2, s[r], b[c][r]) - of.x);
                    ds[c][r] = p[r] * (dp[r] - of.y);
                    most = fmaxf(most, fabsf(ds[c][r]));
                }
                wp[c].set(p);
            }
            if constexpr (kShift<T> != 0.f) {
                const int lifted = lift(group_max(most)), both = lifted < e ? lifted : e;
                if (c0 > 0) {
                    const float down = __builtin_ldexpf(1.f, both - e);
                    ak[0] *= down;
                    ak[1] *= down;
                }
                e = both;
            } else {
                e = 0;
            }
            const float up = __builtin_ldexpf(1.f, e);
#pragma unroll
            for (int c = 0; c < NBLK; ++c) {
                const float t[4] = {ds[c][0] * up, ds[c][1] * up, ds[c][2] * up, ds[c][3] * up};
                ws[c].set(t);
            }
            weighted_sum<T, NBLK>(vector_addr(img_q + kQueryImage, pos, j, g), wp, av);
            weighted_sum<T, NBLK>(vector_addr(img_q, pos, j, g), ws, ak);
        }
        settle_products<2>(ak);
        settle_products<2>(av);
        const float back_v = __builtin_ldexpf(1.f, (int)-kShift<T>), back_k = scale * __builtin_ldexpf(1.f, -e - (int)kShift<T>);
        float xk[8], xv[8], odd = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            xk[d] = ak[d >> 2][d & 3] * back_k;
            xv[d] = av[d >> 2][d & 3] * back_v;
            odd = __builtin_fmaf(xk[d], 0.f, __builtin_fmaf(xv[d], 0.f, odd));
        }
        const unsigned again = marked_columns(odd != odd);
        if (j0 + j >= L) continue;
        if ((again >> j) & 1u) {
            VecN<T, 8> own[2];
            load_vec32(own[0], k + (first + key) * kHeadDim + 8 * g);
            load_vec32(own[1], v + (first + key) * kHeadDim + 8 * g);
            const int i0 = inv_first(key, L, K), at = img_q + (i0 - h0q) * kBytes + g * 16;
            key_once_more<T>(own, at, at + kQueryImage, ld0 + (i0 - h0q) * 8, bias + (key - i0 + K - 1), scale, inv_last(key, L, K) - i0 + 1, xk, xv);
        }
        store_vector<T>(reinterpret_cast<char *>(dk) + (first + key) * kBytes + g * 16, xk);
        store_vector<T>(reinterpret_cast<char *>(dv) + (first + key) * kBytes + g * 16, xv);
    }
}

template <typename T>
hipError_t launch_whole(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, const float *lse, const void *dout,
                        void *dq, void *dk, void *dv, long long *partial, BiasOut d_rpb, hipStream_t s) {
    auto kern = bwd1d_whole_kernel<T>;
    static LdsAllowed allowed;
    if (hipError_t e = allow_lds(kern, whole_lds(kWholeK), allowed); e != hipSuccess) return e;
    const int tiles = (p.L + kWholeTile - 1) / kWholeTile;
    hipLaunchKernelGGL(kern, dim3(p.planes() * tiles), dim3(kWholeThreads), whole_lds(p.K), s, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                       static_cast<const T *>(rpb), scale, lse, static_cast<const T *>(dout), static_cast<T *>(dq), static_cast<T *>(dk), static_cast<T *>(dv), partial,
                       p.L, p.heads, p.K, tiles);
    if (hipError_t e = hipGetLastError(); e != hipSuccess || !d_rpb) return e;
    return launch_rpb_final(RpbTables{partial, d_rpb, p.B, p.heads, tiles, 2 * p.K - 1}, s);
}

// One kernel or two, by their workgroups: the one kernel has 512 places (two to a compute unit), the key side of the two 768 (three).  us of the call, fp16, k = 7, one kernel / two:
// - up to a round of the one kernel: 256 sequences of 250 17.9 / 18.4, 128 of 896 18.2 / 19.0, 16 of 4096 17.6 / 18.3;
// - sequences of 225 to 256, one tile or two: 300 of 226 20.5 / 18.4, 512 of 250 26.0 / 19.0, 1024 of 226 45.6 / 30.6, 2048 of 250 78.7 / 65.0, 4096 of 225 160 / 105, of 256 152 / 126;
// - fewer tiles of 256, in one round: 128 of 1024 22.3 / 19.0, of 1200 23.6 / 21.3, of 1400 27.0 / 22.5, 256 of 490 22.0 / 19.0, 32 of 6000 27.9 / 23.4; more than one: 128 of 1600 30.1 / 29.0, of
//   1900 32.5 / 34.0, 32 of 9000 37.0 / 40.5, 640 of 490 41.7 / 43.5, 4096 of 449 224 / 258;
// - as many of either: 576 of 100 18.3 / 19.0, of 224 20.8 / 20.8, 704 of 224 22.0 / 21.0, 1024 of 200 27.4 / 27.4, 4096 of 224 82 / 102, of 288 159 / 212.
bool one_kernel(const Problem &p) {
    if (p.K > kWholeK) return false;
    const long long one = (long long)p.planes() * ((p.L + kWholeTile - 1) / kWholeTile), two = (long long)p.planes() * ((p.L + kTile - 1) / kTile);
    return launch_holds(one, kWholeThreads) && (one <= 512 || (one < 2 * two && (one == two || two > 768)));
}

template <typename T, typename... Args> hipError_t launch_blocks(const Problem &p, Args... args) {
    switch ((p.K + 15 + 15) / 16) {   // (k from 3 to 63)
        case 2: return launch_t<T, 2>(p, args...);
        case 3: return launch_t<T, 3>(p, args...);
        case 4: return launch_t<T, 4>(p, args...);
        case 5: return launch_t<T, 5>(p, args...);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fused_bwd_16bit(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, const float *lse, const void *dout,
                                  void *dq, void *dk, void *dv, float *delta, long long *partial, BiasOut d_rpb, hipStream_t s) {
    // one kernel: its tables, one per kWholeTile positions, lie from the workspace's first byte on (where the two kernels keep delta, which is no smaller than
    // what they are more than one per 256 positions)
    if (one_kernel(p)) {
        long long *tables = partial ? reinterpret_cast<long long *>(delta) : nullptr;
        return p.dtype == NA2D_F16 ? launch_whole<f16_t>(p, q, k, v, rpb, scale, lse, dout, dq, dk, dv, tables, d_rpb, s)
                                   : launch_whole<bf16_t>(p, q, k, v, rpb, scale, lse, dout, dq, dk, dv, tables, d_rpb, s);
    }
    return p.dtype == NA2D_F16 ? launch_blocks<f16_t>(p, q, k, v, rpb, scale, lse, dout, dq, dk, dv, delta, partial, d_rpb, s)
                               : launch_blocks<bf16_t>(p, q, k, v, rpb, scale, lse, dout, dq, dk, dv, delta, partial, d_rpb, s);
}

}  // namespace na1d
