// The steps without a contraction for window sides beyond the tuned ones (odd K from 15 up to kMaxGenericK): softmax,
// its backward, the bias gradient and the index tables (arXiv 2204.07143, Eq. 4 and the gradients of Appendix A) with
// the window side as a run-time argument, fp32 arithmetic, any of the three storage types.
#include "na2d_kernels.hpp"
#include "na2d_common.hpp"

namespace na2d {

namespace {

struct GShape {
    int H, W, K;
};

// fp32 value of element i of a head vector / row stored as T
template <typename T> __device__ __forceinline__ float ld(const T *p, size_t i) { return to_f32(p[i]); }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// The rows of a workgroup of four waves: WPR waves share a row, NPL values a lane, which stay in registers between the
// reductions and the store.  One wave up to 1024 elements (k = 31), four beyond: with one, 32 and 64 values a lane left
// one to three waves per SIMD.  Measured in 16 bit, us, loop over memory / one wave, loads behind conditions / as here:
// k = 21, 5 x 2 x 64 x 64 rows, softmax 35 / 22 / 13, backward 26 / 28 / 13; k = 45, 2 x 64 x 64 rows, 35 / 19 / 13 and
// 25 / 39 / 12; k = 63, 2 x 63 x 70 rows, 100 / 75 / 23 and 73 / 115 / 22 (5 TB/s).
constexpr int kRowWaves = 4;
template <int WPR> struct RowWave {
    static_assert(WPR == 1 || WPR == kRowWaves);
    size_t row;
    int first;   // the lane's first element; the others follow WPR * kWave apart
    __device__ __forceinline__ RowWave() {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        row = (size_t)blockIdx.x * (kRowWaves / WPR) + wave / WPR;
        first = (wave % WPR) * kWave + threadIdx.x % kWave;
    }
    __device__ __forceinline__ int at(int t) const { return first + t * WPR * kWave; }
    // Past the row's end a lane reads its last element again (the caller drops it): no load is behind a condition, where
    // the conversion of a 16-bit element would wait for its own load, so all of them are in flight at once.
    template <typename T> __device__ __forceinline__ T load(const T *r, int t, int KK) const {
        return r[(unsigned)(at(t) < KK ? at(t) : KK - 1)];
    }
};
// the waves' values of a row, joined in wave order; every wave has read its part of the row before this returns
template <int WPR, typename Op> __device__ __forceinline__ float join_row(float v, float *lds, Op op) {
    if constexpr (WPR == 1) return v;
    else {
        if (threadIdx.x % kWave == 0) lds[threadIdx.x / kWave] = v;
        workgroup_sync();
        float r = lds[0];
#pragma unroll
        for (int w = 1; w < WPR; ++w) r = op(r, lds[w]);
        return r;
    }
}

// softmax of a row (max-subtracted, fp32); out may alias in: the whole row is read before any of it is written
template <typename T, int NPL, int WPR>
__global__ __launch_bounds__(kRowWaves *kWave) void softmax_generic_kernel(const T *in, T *out, int KK, size_t nrows) {
    __shared__ float maxima[kRowWaves], sums[kRowWaves];
    const RowWave<WPR> rw;
    if (rw.row >= nrows) return;   // (with WPR = 4 the same for all waves)
    const T *r = in + rw.row * KK;
    T raw[NPL];
#pragma unroll
    for (int t = 0; t < NPL; ++t) raw[t] = rw.load(r, t, KK);
    float x[NPL], m = -INFINITY;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {
        x[t] = rw.at(t) < KK ? to_f32(raw[t]) : -INFINITY;
        m = fmaxf(m, x[t]);
    }
    m = join_row<WPR>(wave_max(m), maxima, [](float a, float b) { return fmaxf(a, b); });
    float l = 0.f;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {
        x[t] = rw.at(t) < KK ? __expf(x[t] - m) : 0.f;
        l += x[t];
    }
    l = join_row<WPR>(wave_sum(l), sums, [](float a, float b) { return a + b; });
    const float inv = 1.f / l;
    T *o = out + rw.row * KK;
#pragma unroll
    for (int t = 0; t < NPL; ++t)
        if (rw.at(t) < KK) o[(unsigned)rw.at(t)] = from_f32<T>(x[t] * inv);
}

// ds = attn * (dp - <attn, dp>), likewise; ds may alias dp
template <typename T, int NPL, int WPR>
__global__ __launch_bounds__(kRowWaves *kWave) void softmax_bwd_generic_kernel(const T *attn, const T *dp, T *ds, int KK, size_t nrows) {
    __shared__ float dots[kRowWaves];
    const RowWave<WPR> rw;
    if (rw.row >= nrows) return;
    T p[NPL], d[NPL];
    const T *pr = attn + rw.row * KK, *dr = dp + rw.row * KK;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {   // (by turns: all of p before all of d took 281 us instead of 255 in fp32, k = 63)
        p[t] = rw.load(pr, t, KK);
        d[t] = rw.load(dr, t, KK);
    }
    float dot = 0.f;
#pragma unroll
    for (int t = 0; t < NPL; ++t)
        if (rw.at(t) < KK) dot = __builtin_fmaf(to_f32(p[t]), to_f32(d[t]), dot);
    dot = join_row<WPR>(wave_sum(dot), dots, [](float a, float b) { return a + b; });
    T *o = ds + rw.row * KK;
#pragma unroll
    for (int t = 0; t < NPL; ++t)
        if (rw.at(t) < KK) o[(unsigned)rw.at(t)] = from_f32<T>(to_f32(p[t]) * (to_f32(d[t]) - dot));
}

// Bias gradient, first level: one partial table per (plane, range of query rows), one thread per cell (u, v), the
// queries whose window puts a slot on that cell walked in raster order.  The chain of loads along a map row is what
// bounds it, so a row's loads do not depend on each other (a query without such a slot reads one of its own and adds
// nothing), and the rows of a plane are cut into `groups` ranges that run side by side.
template <typename T>
__global__ __launch_bounds__(256) void rpb_generic_partial_kernel(const T *__restrict__ ds, float *__restrict__ partial, GShape g, int groups) {
    const int NB = 2 * g.K - 1, cells = NB * NB, KK = g.K * g.K;
    const int cell_blocks = (cells + 255) / 256;
    const int unit = blockIdx.x / cell_blocks, plane = unit / groups, grp = unit - plane * groups;
    const int cell = (int)(blockIdx.x - unit * cell_blocks) * 256 + threadIdx.x;
    if (cell >= cells) return;
    const int u = cell / NB, vv = cell - u * NB;
    const int row0 = (int)((long long)g.H * grp / groups), row1 = (int)((long long)g.H * (grp + 1) / groups);
    float acc = 0.f;
    for (int qy = row0; qy < row1; ++qy) {
        const int a = u - rpb_start(qy, g.H, g.K);
        if ((unsigned)a >= (unsigned)g.K) continue;
        const T *row = ds + ((size_t)plane * g.H + qy) * g.W * KK + a * g.K;
#pragma unroll 8
        for (int qx = 0; qx < g.W; ++qx) {
            const int c = vv - rpb_start(qx, g.W, g.K), cc = c < 0 ? 0 : (c < g.K ? c : g.K - 1);
            const float v = ld(row, (size_t)qx * KK + cc);
            acc += cc == c ? v : 0.f;
        }
    }
    partial[(size_t)unit * cells + cell] = acc;
}
// second level: 64 cells of a head per workgroup; wave w adds the partials w, w + 16, ... of the head (plane by plane,
// row range by row range), then the 16 sums are added in wave order
constexpr int kFinalWaves = 16;
__global__ __launch_bounds__(kFinalWaves *kWave) void rpb_generic_final_kernel(const float *__restrict__ partial, BiasOut d_rpb,
                                                                               int B, int heads, int cells, int groups) {
    __shared__ float sums[kFinalWaves][kWave];
    const int blocks = (cells + kWave - 1) / kWave, h = blockIdx.x / blocks;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, cell = (blockIdx.x - h * blocks) * kWave + lane;
    float acc = 0.f;
    if (cell < cells) {
#pragma unroll 4
        for (int i = wave; i < B * groups; i += kFinalWaves) {
            const int b = i / groups;
            acc += partial[(((size_t)b * heads + h) * groups + (i - b * groups)) * cells + cell];
        }
    }
    sums[wave][lane] = acc;
    workgroup_sync();
    if (wave == 0 && cell < cells) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < kFinalWaves; ++w) t += sums[w][lane];
        d_rpb.store((size_t)h * cells + cell, t);
    }
}

__global__ __launch_bounds__(256) void indices_generic_kernel(int32_t *key_index, int32_t *rpb_index, int H, int W, int K) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int KK = K * K, NB = 2 * K - 1;
    if (i >= H * W * KK) return;
    const int slot = i % KK, qlin = i / KK;
    const int qy = qlin / W, qx = qlin % W;
    const int a = slot / K, c = slot % K;
    if (key_index) key_index[i] = (win_start(qy, H, K) + a) * W + win_start(qx, W, K) + c;
    if (rpb_index) rpb_index[i] = (rpb_start(qy, H, K) + a) * NB + (rpb_start(qx, W, K) + c);
}

GShape shape_of(const Problem &p) { return GShape{p.H, p.W, p.K}; }

}  // namespace

bool untuned_window(const Problem &p) { return p.K > kMaxTunedK; }

// values a lane keeps of a row: 4 for k = 15, 8 to k = 21, 16 to k = 31; of a quarter of it 8 to k = 45, 16 to k = 63
template <typename T, int NPL = 4, int WPR = 1>
static hipError_t launch_softmax_generic_t(const Problem &p, const T *in, const T *dp, T *out, hipStream_t s) {
    const int KK = p.K * p.K;
    if constexpr (NPL < 16) {
        if (KK > NPL * WPR * kWave) return launch_softmax_generic_t<T, 2 * NPL, WPR>(p, in, dp, out, s);
    } else if constexpr (WPR == 1) {
        if (KK > NPL * kWave) return launch_softmax_generic_t<T, 8, kRowWaves>(p, in, dp, out, s);
    }
    static_assert(kMaxGenericK * kMaxGenericK <= 16 * kRowWaves * kWave);
    const size_t rows = p.queries();
    const dim3 grid((unsigned)((rows * WPR + kRowWaves - 1) / kRowWaves)), block(kRowWaves * kWave);
    if (dp) hipLaunchKernelGGL((softmax_bwd_generic_kernel<T, NPL, WPR>), grid, block, 0, s, in, dp, out, KK, rows);
    else hipLaunchKernelGGL((softmax_generic_kernel<T, NPL, WPR>), grid, block, 0, s, in, out, KK, rows);
    return hipGetLastError();
}

hipError_t launch_softmax_generic(const Problem &p, const void *in, void *out, hipStream_t s) {
    NA2D_DISPATCH_T(p.dtype, return launch_softmax_generic_t<T>(p, static_cast<const T *>(in), nullptr, static_cast<T *>(out), s));
    return hipErrorInvalidValue;
}

hipError_t launch_softmax_bwd_generic(const Problem &p, const void *attn, const void *dp, void *ds, hipStream_t s) {
    NA2D_DISPATCH_T(p.dtype, return launch_softmax_generic_t<T>(p, static_cast<const T *>(attn), static_cast<const T *>(dp), static_cast<T *>(ds), s));
    return hipErrorInvalidValue;
}

// Row ranges per plane: about 4096 workgroups, at most one range per row, and no more partials than the library's own
// scratch array holds (one range always stays allowed), so that the entry point without a workspace takes what it took
// and adds in the same order.
static int rpb_generic_groups(const Problem &p) {
    const int nb = 2 * p.K - 1, cells = nb * nb;
    const long long units = (long long)p.planes() * ((cells + 255) / 256);
    long long n = (4096 + units - 1) / units;
    const long long fit = (long long)NA2D_NOALLOC_SCRATCH_BYTES / ((long long)p.planes() * cells * (long long)sizeof(float));
    n = n < p.H ? n : p.H;
    n = n < fit ? n : fit;
    return n < 1 ? 1 : (int)n;
}

size_t rpb_generic_workspace_bytes(const Problem &p) {
    const int nb = 2 * p.K - 1;
    return (size_t)p.planes() * rpb_generic_groups(p) * nb * nb * sizeof(float);
}

hipError_t launch_rpb_generic(const Problem &p, const void *ds, BiasOut d_rpb, void *workspace, hipStream_t s) {
    const int nb = 2 * p.K - 1, cells = nb * nb, groups = rpb_generic_groups(p);
    NA2D_DISPATCH_T(p.dtype, hipLaunchKernelGGL((rpb_generic_partial_kernel<T>), dim3((unsigned)(((cells + 255) / 256) * (size_t)p.planes() * groups)), dim3(256), 0, s,
                                                static_cast<const T *>(ds), static_cast<float *>(workspace), shape_of(p), groups));
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    hipLaunchKernelGGL(rpb_generic_final_kernel, dim3(p.heads * ((cells + kWave - 1) / kWave)), dim3(kFinalWaves * kWave), 0, s,
                       static_cast<const float *>(workspace), d_rpb, p.B, p.heads, cells, groups);
    return hipGetLastError();
}

hipError_t launch_indices_generic(const Problem &p, int32_t *key_index, int32_t *rpb_index, hipStream_t s) {
    const int n = p.H * p.W * p.K * p.K;
    hipLaunchKernelGGL(indices_generic_kernel, dim3((n + 255) / 256), dim3(256), 0, s, key_index, rpb_index, p.H, p.W, p.K);
    return hipGetLastError();
}

}  // namespace na2d
