// The steps without a contraction for window sides beyond the tuned ones (odd K from 15 up to kMaxGenericK): softmax,
// its backward, the bias gradient and the index tables (arXiv 2204.07143, Eq. 4 and the gradients of Appendix A) with
// the window side as a run-time argument, fp32 arithmetic, any of the three storage types.
#include "na2d_kernels.hpp"
#include "na2d_common.hpp"

namespace na2d {

namespace {

struct GShape {
    int B, heads, H, W, K, D;
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

// Softmax of one row per wave (max-subtracted, fp32).  The row stays in registers, NPL values a lane, between the
// maximum, the sum and the store; out may alias in: the whole row is read before any of it is written.
template <typename T, int NPL>
__global__ __launch_bounds__(256) void softmax_generic_kernel(const T *in, T *out, int KK, size_t nrows) {
    const size_t row = (size_t)blockIdx.x * 4 + threadIdx.x / kWave;
    const int lane = threadIdx.x % kWave;
    if (row >= nrows) return;
    const T *r = in + row * KK;
    float x[NPL], m = -INFINITY;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {
        const int i = lane + t * kWave;
        x[t] = i < KK ? ld(r, i) : -INFINITY;
        m = fmaxf(m, x[t]);
    }
    m = wave_max(m);
    float l = 0.f;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {
        x[t] = lane + t * kWave < KK ? __expf(x[t] - m) : 0.f;
        l += x[t];
    }
    l = wave_sum(l);
    const float inv = 1.f / l;
    T *o = out + row * KK;
#pragma unroll
    for (int t = 0; t < NPL; ++t)
        if (lane + t * kWave < KK) o[lane + t * kWave] = from_f32<T>(x[t] * inv);
}

// ds = attn * (dp - <attn, dp>), one row per wave, in registers likewise; ds may alias dp
template <typename T, int NPL>
__global__ __launch_bounds__(256) void softmax_bwd_generic_kernel(const T *attn, const T *dp, T *ds, int KK, size_t nrows) {
    const size_t row = (size_t)blockIdx.x * 4 + threadIdx.x / kWave;
    const int lane = threadIdx.x % kWave;
    if (row >= nrows) return;
    const T *pr = attn + row * KK, *dr = dp + row * KK;
    float p[NPL], d[NPL], dot = 0.f;
#pragma unroll
    for (int t = 0; t < NPL; ++t) {
        const int i = lane + t * kWave;
        p[t] = i < KK ? ld(pr, i) : 0.f;
        d[t] = i < KK ? ld(dr, i) : 0.f;
    }
#pragma unroll
    for (int t = 0; t < NPL; ++t) dot = __builtin_fmaf(p[t], d[t], dot);
    dot = wave_sum(dot);
    T *o = ds + row * KK;
#pragma unroll
    for (int t = 0; t < NPL; ++t)
        if (lane + t * kWave < KK) o[lane + t * kWave] = from_f32<T>(p[t] * (d[t] - dot));
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
__global__ __launch_bounds__(kFinalWaves *kWave) void rpb_generic_final_kernel(const float *__restrict__ partial, float *__restrict__ d_rpb,
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
        d_rpb[(size_t)h * cells + cell] = t;
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

GShape shape_of(const Problem &p) { return GShape{p.B, p.heads, p.H, p.W, p.K, p.D}; }

}  // namespace

bool untuned_window(const Problem &p) { return p.K > kMaxTunedK; }

// values a lane keeps of a row, rounded up to a power of two: 4 for K = 15 up to 64 for K = 63
template <typename T, int NPL = 4>
static hipError_t launch_softmax_generic_t(const Problem &p, const T *in, const T *dp, T *out, hipStream_t s) {
    const int KK = p.K * p.K;
    if constexpr (NPL < 64)
        if (KK > NPL * kWave) return launch_softmax_generic_t<T, 2 * NPL>(p, in, dp, out, s);
    const size_t rows = p.queries();
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    if (dp) hipLaunchKernelGGL((softmax_bwd_generic_kernel<T, NPL>), grid, block, 0, s, in, dp, out, KK, rows);
    else hipLaunchKernelGGL((softmax_generic_kernel<T, NPL>), grid, block, 0, s, in, out, KK, rows);
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

hipError_t launch_rpb_generic(const Problem &p, const void *ds, float *d_rpb, void *workspace, hipStream_t s) {
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
