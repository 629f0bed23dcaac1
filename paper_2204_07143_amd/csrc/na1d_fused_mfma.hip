// Fused 1D neighbourhood attention forward on the matrix cores, f16 / bf16 (arXiv 2204.07143, Section 3.1, Eq. 2-4 on a sequence).
//
// The windows of 16 consecutive queries reach 16 + k - 1 consecutive keys: NBLK = ceil((k + 15) / 16) blocks of 16, counted from the first
// query's window, hold them (2 to 5 for k = 3 .. 63).  Per group of 16 queries
//   S^T = K_blk Q^T                 one full-depth MFMA per block (a lane holds four keys of its query)
//   P = exp2(S' + bias - max)       the bias, -inf outside the window, stays in registers: it is the same for every group
//                                   whose windows are clear of the sequence's ends
//   out^T += V_blk^T P              values through the transposing LDS read
// P enters the product as two 16-bit halves, its value rounded and the rounding's remainder, so that it counts with 22 (fp16) or 16 (bf16)
// digits; in fp16 it is scaled by 2^15 first, for the remainder not to fall below the type's smallest numbers.
// A workgroup of four waves keeps 64 GPW queries; the keys and values they reach go to LDS by direct loads, all at once.  One group per
// wave (GPW 1) is for calls whose tiles of four would not fill the chip.
// A masked product is 0 * x: where a value is not finite it would spoil queries whose window does not hold it, so results that are not
// finite are computed once more from their own window.
// Bound by memory: 64 x 2 x 3136 queries (103 MB) take 18.7 us in fp16 at k = 7, 19.7 us in bf16 at k = 31 and 23.5 us at k = 63, 4.4 to
// 5.5 TB/s; a thread per query with its products on the plain ALU took 24.6, 51.2 and 105 us.
#include "lds_attr.hpp"
#include "na1d_common.hpp"
#include "na1d_kernels.hpp"

namespace na1d {

using namespace na2d;

namespace {

constexpr int kWaves = 4, kThreads = kWaves * kWave;

template <int NBLK, int GPW> struct Cfg {
    static constexpr int TQ = kWaves * GPW * kGroup, ROWS = TQ - kGroup + 16 * NBLK;   // queries, keys staged
    static constexpr int kImage = ROWS * kBytes;
    static constexpr int kLds = 2 * kImage;   // and 2 K - 1 floats of bias
};

// One query from its own window, as plain sums: lane group g keeps channels 8 g .. 8 g + 7.  An lse that is finite stays.  (What is NaN stays NaN:
// the rest of the window is left out.)  ka, va: this lane's part of the window's first key and value in LDS; bias: of the window's first slot.
template <typename T>
__device__ void query_once_more(const u32x4 &own, int ka, int va, const float *bias, float scale2, int K, float (&acc)[8], float &lse) {
    VecN<T, 8> qv;   // (the four lanes of a column work on it, eight channels each)
    qv.w[0] = own.x, qv.w[1] = own.y, qv.w[2] = own.z, qv.w[3] = own.w;
    float m = kLowest, l = 0.f;
    const bool keep = fabsf(lse) < INFINITY;
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] = 0.f;
#pragma unroll 1
    for (int a = 0; a < K; a += kOnceMore) {
        float s[kOnceMore], most = m;
        VecN<T, 8> v[kOnceMore];
#pragma unroll
        for (int e = 0; e < kOnceMore; ++e) {
            const int at = a + e < K ? a + e : K - 1;   // (past the end: once more, not added)
            VecN<T, 8> kv;
            load8_lds(kv, ka + at * kBytes);
            load8_lds(v[e], va + at * kBytes);
            s[e] = __builtin_fmaf(scale2, group_sum(dot32(qv, kv)), bias[at]);
            most = fmaxf(most, s[e]);
        }
        const float c = __builtin_amdgcn_exp2f(m - most);
        m = most;
        l *= c;
#pragma unroll
        for (int d = 0; d < 8; ++d) acc[d] *= c;
#pragma unroll
        for (int e = 0; e < kOnceMore; ++e)
            if (a + e < K) {
                const float p = __builtin_amdgcn_exp2f(s[e] - m);
                l += p;
                axpy32(acc, p, v[e]);
            }
        float open = keep ? 0.f : 1.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) open = acc[d] == acc[d] ? 1.f : open;
        if (l != l || group_sum(open) == 0.f) break;
    }
    if (l == 0.f) l = NAN;   // every logit -inf
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] *= 1.f / l;
    if (!keep) lse = (m + __builtin_amdgcn_logf(l)) * kLn2;
}

template <typename T, int NBLK, int GPW>
__global__ __launch_bounds__(kThreads, 4) void fused1d_mfma_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
                                                                   const T *__restrict__ rpb, float scale, T *__restrict__ out,
                                                                   float *__restrict__ lse, int L, int heads, int K, int tiles) {
    using C = Cfg<NBLK, GPW>;
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave), j = lane & 15, g = lane >> 4;
    const int plane = blockIdx.x / tiles, t0 = (blockIdx.x - plane * tiles) * C::TQ, NB = 2 * K - 1;
    const size_t first = (size_t)plane * L;
    const int h0 = win_start(t0, L, K), img = lds_addr(lds);
    float *bias = reinterpret_cast<float *>(lds + C::kLds);

    stage_pair<kWaves>(reinterpret_cast<const char *>(k) + (first + h0) * kBytes, reinterpret_cast<const char *>(v) + (first + h0) * kBytes, L - 1 - h0,
                       C::ROWS, img, img + C::kImage, wave, lane);
    u32x4 qv[GPW];
#pragma unroll
    for (int n = 0; n < GPW; ++n) {
        const int i = t0 + (wave * GPW + n) * kGroup + j;
        qv[n] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(q) + (first + (i < L ? i : L - 1)) * kBytes + g * 16);
    }
    const T *table = rpb ? rpb + (size_t)(plane % heads) * NB : nullptr;
    for (int u = tid; u < NB; u += kThreads) bias[u] = table ? to_f32(table[u]) * kLog2e : 0.f;
    wait_global_loads();
    workgroup_sync();

    const float scale2 = scale * kLog2e;
    float b[NBLK][4];
    bool inner = false;   // b[] is that of a group clear of the ends
#pragma unroll
    for (int n = 0; n < GPW; ++n) {
        const int i0 = t0 + (wave * GPW + n) * kGroup;
        if (i0 >= L) break;
        const int o = win_start(i0, L, K), i = i0 + j < L ? i0 + j : L - 1;
        const bool clear = o == i0 - (K >> 1) && i0 + kGroup - 1 + (K >> 1) < L;
        if (!(clear && inner)) {
            const int w = win_start(i, L, K) - o;   // the lane's window begins at position w of the blocks
#pragma unroll
            for (int c = 0; c < NBLK; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = 16 * c + 4 * g + r;
                    const bool in = (unsigned)(at - w) < (unsigned)K;
                    const float t = bias[in ? at + o - i + K - 1 : 0];
                    b[c][r] = in ? t : -INFINITY;
                }
            inner = clear;
        }
        const int kaddr = row_addr(img, o - h0, j, g);
        f32x4 s[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) s[c] = mfma_16x16x32<T>(*lds_ptr<u32x4>(kaddr + c * 1024), qv[n], f32x4{0.f, 0.f, 0.f, 0.f});
        float m = -INFINITY;
#pragma unroll
        for (int c = 0; c < NBLK; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] = __builtin_fmaf(scale2, s[c][r], b[c][r]);
                m = fmaxf(m, s[c][r]);
            }
        m = group_max(m) - kShift<T>;
        float l = 0.f;
        Split4<T> w[NBLK];
#pragma unroll
        for (int c = 0; c < NBLK; ++c) {
            float p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = __builtin_amdgcn_exp2f(s[c][r] - m);
                l += p[r];
            }
            w[c].set(p);
        }
        l = group_sum(l);
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        weighted_sum<T, NBLK>(vector_addr(img + C::kImage, o - h0, j, g), w, acc);
        const float inv = 1.f / l;
        float x[8], log_sum = (m + __builtin_amdgcn_logf(l)) * kLn2, odd = log_sum * 0.f;   // odd: NaN where something is not finite
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            x[d] = acc[d >> 2][d & 3] * inv;
            odd = __builtin_fmaf(x[d], 0.f, odd);
        }
        const unsigned again = marked_columns(odd != odd);
        if ((again >> j) & 1u) {
            const int s0 = win_start(i, L, K), ka = img + (s0 - h0) * kBytes + g * 16;
            query_once_more<T>(qv[n], ka, ka + C::kImage, bias + (s0 - i + K - 1), scale2, K, x, log_sum);
        }
        if (i0 + j < L) {
            store_vector<T>(reinterpret_cast<char *>(out) + (first + i) * kBytes + g * 16, x);
            if (lse != nullptr && g == 0) lse[first + i] = log_sum;
        }
    }
}

template <typename T, int NBLK, int GPW>
hipError_t launch_t(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, void *out, float *lse, hipStream_t s) {
    using C = Cfg<NBLK, GPW>;
    auto kern = fused1d_mfma_kernel<T, NBLK, GPW>;
    constexpr int kMost = C::kLds + (2 * kMaxK - 1) * 4;
    static LdsAllowed allowed;
    if (hipError_t e = allow_lds(kern, kMost, allowed); e != hipSuccess) return e;
    const int tiles = (p.L + C::TQ - 1) / C::TQ;
    hipLaunchKernelGGL(kern, dim3(p.planes() * tiles), dim3(kThreads), C::kLds + (2 * p.K - 1) * 4, s, static_cast<const T *>(q),
                       static_cast<const T *>(k), static_cast<const T *>(v), static_cast<const T *>(rpb), scale, static_cast<T *>(out), lse,
                       p.L, p.heads, p.K, tiles);
    return hipGetLastError();
}

template <typename T, int NBLK>
hipError_t launch_groups(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, void *out, float *lse, hipStream_t s) {
    // four groups to a wave stage 64 GPW + 16 NBLK - 16 keys for 64 GPW queries where one group stages twice what it needs and more; from two
    // tiles per compute unit on that counts more than the longer chain of a wave (small calls are below the launch's own time either way)
    const size_t tiles = (size_t)p.planes() * ((p.L + 4 * kWaves * kGroup - 1) / (4 * kWaves * kGroup));
    return tiles >= 512 ? launch_t<T, NBLK, 4>(p, q, k, v, rpb, scale, out, lse, s) : launch_t<T, NBLK, 1>(p, q, k, v, rpb, scale, out, lse, s);
}

template <typename T>
hipError_t launch_blocks(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, void *out, float *lse, hipStream_t s) {
    switch ((p.K + 15 + 15) / 16) {   // (k from 3 to 63)
        case 2: return launch_groups<T, 2>(p, q, k, v, rpb, scale, out, lse, s);
        case 3: return launch_groups<T, 3>(p, q, k, v, rpb, scale, out, lse, s);
        case 4: return launch_groups<T, 4>(p, q, k, v, rpb, scale, out, lse, s);
        case 5: return launch_groups<T, 5>(p, q, k, v, rpb, scale, out, lse, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fused_fwd_16bit(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, void *out,
                                  float *lse, hipStream_t s) {
    return p.dtype == NA2D_F16 ? launch_blocks<f16_t>(p, q, k, v, rpb, scale, out, lse, s) : launch_blocks<bf16_t>(p, q, k, v, rpb, scale, out, lse, s);
}

}  // namespace na1d
