// Neighbourhood attention on the matrix cores for any window side and any storage type, fp32 included (arXiv
// 2204.07143, Eq. 2-4 and the gradients of Appendix A): the contractions of the problems that have no kernel of a
// fixed window side.
//
// A strip is 16 consecutive positions of one map row; a workgroup's four waves take its window rows in turn, or a strip each.
// For one window row the strip's windows together cover 16 + K - 1 consecutive positions of one row of the other
// operand, i.e. one small dense product of 16 strip positions with blocks of 16 partner positions, masked by the
// window.  Nothing but the waves' partial sums is staged in LDS, so neither the window nor the head dim is limited
// by it: partner positions come from global memory (neighbouring strips re-read them out of L2), the weights are
// read or written in place (a 4 x 4 patch would have fewer masked products, but its weights do not lie in one run per row).
// What bounds it, by counters at 4 x 2 x 64 x 64 x 32, k = 21, bf16 (107520 blocks of 16 x 16 products): the logits (41 us)
// their 430k stores, two bytes a lane, 59 % of the wave cycles waiting; the weighted sums (44 us, inverse 26) 8 loads per block, 67
// and 54 % waiting; the fused forward (50 us; such calls run over the patches of na2d_patch_fwd.hip now) its 188 vector instructions per block, 33 us at
// four cycles each, 20 % waiting.
//
// Measured against one thread per output element (that shape, forward and backward of the fused operator, together with
// the steps of na2d_generic.hip): 3099 -> 268 us.
//
// Weights that are stored are products of 16-bit (or fp32) operands summed in fp32: exact products as on the plain
// ALU.  The fused forward keeps its weights in fp32; in 16 bit they enter as a high and a low half, two products instead
// of one: p = hi + lo to 2^-17 of p in bf16.  In fp16 they are scaled by 2^15 first (kWeightUp; the sum of the weights
// likewise, so that it cancels): then the halves hold p to 2^-22 of itself down to p = 2^-18 of the largest weight and to
// 2^-40 of the largest below, instead of to 2^-25 (below which a weight left the numerator but not the sum).
//
// A masked product is 0 * y.  Where y is not finite that would spoil positions whose window does not hold it, so an
// output that is not finite is computed once more from its own window only, which ends as soon as its sum is NaN.  A call
// on values of NaN then took (us, finite values in brackets; the fused calls run over patches now): fused forward 7 x 100 x 134, D = 128, k = 9, f16 654 (123; a
// thread per output that worked out every logit again: 15400), 4 x 2 x 64 x 64, D = 32, k = 21, bf16 66 (45; 1230); weighted sum there 52 (44; with the whole window 178), inverse 39 (25; 263).
#include <limits.h>

#include "na2d_kernels.hpp"
#include "na2d_mfma.hpp"
#include "na2d_tile.hpp"

namespace na2d {

namespace {

constexpr int kStripWaves = 4, kStripThreads = kStripWaves * kWave;

struct SShape {
    int heads, H, W, K, strips, rows, ntiles;   // strips per map row, rows of workgroups per plane
};

// SPLIT waves share a strip; the kStripWaves / SPLIT strips of a workgroup lie one below the other.
struct Strip {
    int plane, y, x0;
    int wave, part;   // wave of the workgroup, and which of the strip's window rows (part, part + SPLIT, ...) it takes
};
template <int SPLIT> __device__ __forceinline__ bool decode_strip(const SShape &g, Strip &s) {
    const int t = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (t >= g.ntiles) return false;
    s.wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    s.part = s.wave % SPLIT;
    s.x0 = (t % g.strips) * kStrip;
    const int rest = t / g.strips;
    s.y = (rest % g.rows) * (kStripWaves / SPLIT) + s.wave / SPLIT;
    s.plane = rest / g.rows;
    return s.y < g.H;   // (with SPLIT = 4 the same for all waves of a workgroup, which then meet at a barrier)
}
// the waves of a strip have left their sums in LDS
template <int SPLIT> __device__ __forceinline__ void join_waves() {
    if constexpr (SPLIT > 1) {
        workgroup_sync();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <typename T> __device__ __forceinline__ uint32_t pack2(T lo, T hi) {
    return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}
__device__ __forceinline__ f32x4 mfma_16x16x4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// One head vector per 16-lane column, as an operand whose contraction runs over channels.  Lane (column j, group g)
// holds, of each `step` channels, the 16-byte chunk g (both operands alike, so the order of channels is free).
template <typename T, int D> struct ChannelOp {
    static constexpr int EPC = 16 / (int)sizeof(T);            // channels per chunk
    static constexpr int N = (D + 4 * EPC - 1) / (4 * EPC);    // chunks per lane (D = 16 in 16 bit: half the lanes hold zeros)
    u32x4 c[N];
    __device__ __forceinline__ void load(const T *vec, int g) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            c[i] = u32x4{0u, 0u, 0u, 0u};
            if ((4 * i + g) * EPC < D) c[i] = *reinterpret_cast<const u32x4 *>(vec + (4 * i + g) * EPC);
        }
    }
};
// result rows: positions 4 g + r of the first operand; columns: positions of the second
template <typename T, int D>
__device__ __forceinline__ f32x4 dot_block(const ChannelOp<T, D> &a, const ChannelOp<T, D> &b) {
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < ChannelOp<T, D>::N; ++i) {
        if constexpr (sizeof(T) == 4) {
            const f32x4 x = __builtin_bit_cast(f32x4, a.c[i]), y = __builtin_bit_cast(f32x4, b.c[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = mfma_16x16x4(x[e], y[e], acc);
        } else {
            acc = mfma_16x16x32<T>(a.c[i], b.c[i], acc);
        }
    }
    return acc;
}

// The weighted sum of 16 positions, channels as result rows: lane (column j, group g) brings channel(s) j of the
// positions 4 g .. 4 g + 3 and the weights of strip position j for the same four.  Head dims of 32 and more are
// loaded two channels at a time: rows of block 2 p are the even, of block 2 p + 1 the odd channels of slice p.
template <typename T, int D> struct SumAcc {
    static constexpr int NB = D / 16;
    f32x4 acc[NB];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ static __forceinline__ int channel(int block, int row) {
        return D == 16 ? row : (block >> 1) * 32 + 2 * row + (block & 1);
    }
    // NW sets of weights (their sum is meant): w[s][e] for position e
    template <int NW> __device__ __forceinline__ void add(const T *y, const int (&off)[4], int j, const T (&w)[NW][4]) {
        if constexpr (D == 16) {
            T v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = y[off[e] + j];
            product<NW>(acc[0], v, w);
        } else {
#pragma unroll
            for (int p = 0; p < D / 32; ++p) {
                T lo[4], hi[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    struct alignas(2 * sizeof(T)) Pair { T a, b; };
                    const Pair t = *reinterpret_cast<const Pair *>(y + off[e] + p * 32 + 2 * j);
                    lo[e] = t.a;
                    hi[e] = t.b;
                }
                product<NW>(acc[2 * p], lo, w);
                product<NW>(acc[2 * p + 1], hi, w);
            }
        }
    }
    template <int NW> __device__ static __forceinline__ void product(f32x4 &c, const T (&v)[4], const T (&w)[NW][4]) {
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) c = mfma_16x16x4(v[e], w[s][e], c);
            } else {
                c = mfma_16x16x16<T>(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(w[s][0], w[s][1]), pack2(w[s][2], w[s][3]), c);
            }
        }
    }
    // the wave's sums to LDS as [strip position][channel]
    static constexpr int kPitch = D + 1;
    __device__ __forceinline__ void to_lds(float *dst, int j, int g) const {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[j * kPitch + channel(i, 4 * g + r)] = acc[i][r];
    }
};

__device__ __forceinline__ int clamp_to(int v, int hi) { return v < 0 ? 0 : (v < hi ? v : hi); }

// logits[n, a, c] = scale <x_n, y_key(n; a, c)> + bias (and grad-a: x = dout, y = v)
template <typename T, int D, int SPLIT>
__global__ __launch_bounds__(kStripThreads) void qk_strip_kernel(const T *__restrict__ x, const T *__restrict__ y,
                                                                 const T *__restrict__ rpb, float scale, T *__restrict__ logits, SShape g) {
    Strip st;
    if (!decode_strip<SPLIT>(g, st)) return;
    const int lane = threadIdx.x % kWave, j = lane % 16, grp = lane / 16;
    const int K = g.K, W = g.W, KK = K * K, NB = 2 * K - 1;
    const size_t plane0 = (size_t)st.plane * g.H * W;
    const bool mine = st.x0 + j < W;
    const int qx = mine ? st.x0 + j : W - 1, sx = win_start(qx, W, K), sy = win_start(st.y, g.H, K);
    const int kx0 = win_start(st.x0, W, K);
    const int xl = st.x0 + kStrip - 1 < W ? st.x0 + kStrip - 1 : W - 1, nblk = (win_start(xl, W, K) + K - 1 - kx0) / 16 + 1;
    ChannelOp<T, D> xo;
    xo.load(x + (plane0 + (size_t)st.y * W + qx) * D, grp);
    const T *yp = y + plane0 * D;
    T *row = logits + (plane0 + (size_t)st.y * W + qx) * KK;
    const T *bt = rpb ? rpb + ((size_t)(st.plane % g.heads) * NB + (sy - st.y + K - 1)) * NB + (sx - qx + K - 1) : nullptr;
    // The bias entries of a block are loaded beside its keys, not one after the other behind each store's condition (us, before /
    // after: f16, D = 16, k = 15, one 28 x 28 map 4.8 / 4.1; fp32, D = 16, k = 45, 2 x 100 x 134 202 / 135; bf16, D = 32, k = 21,
    // 2 x 64 x 64 13.9 / 12.8).  128 channels in fp32 lose 5 % by it (the registers).
    constexpr bool kBiasFirst = D * sizeof(T) <= 256;
    for (int a = blockIdx.y * SPLIT + st.part; a < K; a += SPLIT * gridDim.y) {
        const T *yrow = yp + (size_t)(sy + a) * W * D;
        for (int b = 0; b < nblk; ++b) {
            const int k0 = kx0 + 16 * b, kl = k0 + j < W ? k0 + j : W - 1;
            ChannelOp<T, D> yo;
            yo.load(yrow + (size_t)kl * D, grp);
            const int c0 = k0 + 4 * grp - sx;
            T bias[4] = {};
            if constexpr (kBiasFirst) {
                if (bt) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) bias[r] = bt[a * NB + clamp_to(c0 + r, K - 1)];   // (outside the window unused)
                }
            }
            const f32x4 s = dot_block<T, D>(yo, xo);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = mine && (unsigned)(c0 + r) < (unsigned)K;
                if constexpr (kBiasFirst) {
                    const float v = bt ? __builtin_fmaf(scale, s[r], to_f32(bias[r])) : scale * s[r];
                    if (in) row[a * K + c0 + r] = from_f32<T>(v);
                } else if (in) {
                    const float v = bt ? __builtin_fmaf(scale, s[r], to_f32(bt[a * NB + c0 + r])) : scale * s[r];
                    row[a * K + c0 + r] = from_f32<T>(v);
                }
            }
        }
    }
}

// One output of the weighted sum from its own window, in raster order (strip outputs that are not finite).  A sum that is
// NaN stays NaN, so the walk ends there: where a whole tensor is NaN (a step that diverged) it reads one window row.
template <typename T, int D, bool INV>
__device__ __noinline__ float sum_one(const T *w, const T *y, int H, int W, int K, int py, int px, int d) {
    const int KK = K * K;
    float acc = 0.f;
    const int y0 = INV ? inv_first(py, H, K) : win_start(py, H, K), y1 = INV ? inv_last(py, H, K) : y0 + K - 1;
    const int x0 = INV ? inv_first(px, W, K) : win_start(px, W, K), x1 = INV ? inv_last(px, W, K) : x0 + K - 1;
    for (int oy = y0; oy <= y1 && acc == acc; ++oy) {
        for (int ox = x0; ox <= x1; ++ox) {
            const size_t n = INV ? (size_t)oy * W + ox : (size_t)py * W + px;
            const int slot = INV ? (py - win_start(oy, H, K)) * K + px - win_start(ox, W, K) : (oy - y0) * K + ox - x0;
            acc = __builtin_fmaf(to_f32(w[n * KK + slot]), to_f32(y[((size_t)oy * W + ox) * D + d]), acc);
        }
    }
    return acc;
}

// INV false: out[n, :] = scale sum_slot w[n, slot] y_key(n; slot).  INV true: out[j, :] = scale sum of w[i, slot(i, j)] y_i
// over the queries i that see key j.  The waves' sums are added in wave order: the same bits in every run.
template <typename T, int D, bool INV, int SPLIT>
__global__ __launch_bounds__(kStripThreads) void sum_strip_kernel(const T *__restrict__ w, const T *__restrict__ y, float scale,
                                                                  T *__restrict__ out, SShape g) {
    using A = SumAcc<T, D>;
    __shared__ float part[kStripWaves][kStrip * A::kPitch];
    Strip st;
    if (!decode_strip<SPLIT>(g, st)) return;
    const int lane = threadIdx.x % kWave, j = lane % 16, grp = lane / 16;
    const int K = g.K, W = g.W, H = g.H, KK = K * K;
    const size_t plane0 = (size_t)st.plane * H * W;
    const T *wp = w + plane0 * KK, *yp = y + plane0 * D;
    const int px = st.x0 + j < W ? st.x0 + j : W - 1;
    const int xl = st.x0 + kStrip - 1 < W ? st.x0 + kStrip - 1 : W - 1;
    const int first = INV ? inv_first(st.x0, W, K) : win_start(st.x0, W, K);
    const int last = INV ? inv_last(xl, W, K) : win_start(xl, W, K) + K - 1;
    const int nblk = (last - first) / 16 + 1;
    const int y0 = INV ? inv_first(st.y, H, K) : win_start(st.y, H, K);
    const int y1 = INV ? inv_last(st.y, H, K) : y0 + K - 1;
    const int sx = win_start(px, W, K);
    A acc;
    acc.clear();
    for (int oy = y0 + st.part; oy <= y1; oy += SPLIT) {
        const int a = INV ? st.y - win_start(oy, H, K) : oy - y0;
        const int wrow = INV ? oy * W * KK + a * K : (st.y * W + px) * KK + a * K;
        for (int b = 0; b < nblk; ++b) {
            T wt[1][4];
            int off[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ox = first + 16 * b + 4 * grp + e, oc = ox < W ? ox : W - 1;
                const int c = INV ? px - win_start(oc, W, K) : ox - sx;
                const bool in = (unsigned)c < (unsigned)K && ox < W;
                const T v = wp[wrow + (INV ? oc * KK : 0) + clamp_to(c, K - 1)];
                wt[0][e] = in ? v : (T)0.f;
                off[e] = (oy * W + oc) * D;
            }
            acc.template add<1>(yp, off, j, wt);
        }
    }
    acc.to_lds(part[st.wave], j, grp);
    join_waves<SPLIT>();
    const int w0 = st.wave - st.part;   // the strip's first wave
    for (int i = st.part * kWave + lane; i < kStrip * D; i += SPLIT * kWave) {
        const int p = i / D, d = i % D;
        if (st.x0 + p >= W) break;   // (p grows with i)
        float v = 0.f;
#pragma unroll
        for (int s = 0; s < SPLIT; ++s) v += part[w0 + s][p * A::kPitch + d];
        if (!(fabsf(v) < INFINITY)) v = sum_one<T, D, INV>(wp, yp, H, W, K, st.y, st.x0 + p, d);
        out[(plane0 + (size_t)st.y * W + st.x0 + p) * D + d] = from_f32<T>(scale * v);
    }
}

// fp32 dot product of two head vectors
template <typename T, int D> __device__ __forceinline__ float dot_one(const T *a, const T *b) {
    float acc = 0.f;
#pragma unroll 8
    for (int d = 0; d < D; ++d) acc = __builtin_fmaf(to_f32(a[d]), to_f32(b[d]), acc);
    return acc;
}
// The fused outputs of one position from its own window, in raster order (strip outputs that are not finite): the whole
// wave works out the weights of 64 slots, a slot to a lane, then each lane adds up its channel d.  `wanted`: the lanes whose
// sum is asked for; once all of them are NaN nothing changes any more.
template <typename T, int D>
__device__ __noinline__ float fused_position(const T *q, const T *kp, const T *vp, const T *bt, float scale, float m, int W, int K, int sy, int sx, int d, bool wanted) {
    constexpr int kAtOnce = 8;
    const int KK = K * K, lane = threadIdx.x % kWave;
    float acc = 0.f;
    int a0 = 0, c0 = 0;   // the chunk's first slot
    for (int first = 0; first < KK; first += kWave) {
        const int slot = first + lane < KK ? first + lane : KK - 1, a = slot / K, c = slot - a * K;
        float s = scale * dot_one<T, D>(q, kp + ((size_t)(sy + a) * W + sx + c) * D);
        if (bt) s += to_f32(bt[a * (2 * K - 1) + c]);
        const float w = __expf(s - m);
        const int n = KK - first < kWave ? KK - first : kWave;
        for (int t = 0; t < n; t += kAtOnce) {   // (their loads do not wait for each other)
            float wt[kAtOnce], y[kAtOnce];
#pragma unroll
            for (int e = 0; e < kAtOnce; ++e) {
                wt[e] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), (t + e) % kWave));
                y[e] = to_f32(vp[((size_t)(sy + a0) * W + sx + c0) * D + d]);
                if (++c0 == K) {   // (past the last slot it stays there: read once more, not added)
                    const bool more = a0 < K - 1;
                    c0 = more ? 0 : K - 1;
                    a0 += more;
                }
            }
#pragma unroll
            for (int e = 0; e < kAtOnce; ++e)
                if (t + e < n) acc = __builtin_fmaf(wt[e], y[e], acc);
            if (__ballot(wanted && acc == acc) == 0) return acc;
        }
    }
    return acc;
}

// the power of two by which the fused forward's weights are scaled: the largest is then 2^15, within fp16's range
template <typename T> constexpr float kWeightUp = 1.f;
template <> constexpr float kWeightUp<f16_t> = 32768.f;

// Fused forward.  Each wave keeps a running maximum, sum and weighted values of its window rows, NBX blocks of 16 keys
// at a time; the logits leave the matrix cores in the layout in which the weights enter them again.  The waves'
// results are joined in wave order.
template <typename T, int D, int NBX, int SPLIT>
__global__ __launch_bounds__(kStripThreads) void fused_strip_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                    const T *__restrict__ v, const T *__restrict__ rpb, float scale,
                                                                    T *__restrict__ out, float *__restrict__ lse, SShape g) {
    using A = SumAcc<T, D>;
    constexpr int NW = sizeof(T) == 4 ? 1 : 2;
    __shared__ float part[kStripWaves][kStrip * A::kPitch];
    __shared__ float wm[kStripWaves][kStrip], wl[kStripWaves][kStrip];
    Strip st;
    if (!decode_strip<SPLIT>(g, st)) return;
    const int lane = threadIdx.x % kWave, j = lane % 16, grp = lane / 16;
    const int K = g.K, W = g.W, NB = 2 * K - 1;
    const size_t plane0 = (size_t)st.plane * g.H * W;
    const int qx = st.x0 + j < W ? st.x0 + j : W - 1, sx = win_start(qx, W, K), sy = win_start(st.y, g.H, K);
    const int kx0 = win_start(st.x0, W, K);
    const int xl = st.x0 + kStrip - 1 < W ? st.x0 + kStrip - 1 : W - 1, nblk = (win_start(xl, W, K) + K - 1 - kx0) / 16 + 1;
    ChannelOp<T, D> qo;
    qo.load(q + (plane0 + (size_t)st.y * W + qx) * D, grp);
    const T *kp = k + plane0 * D, *vp = v + plane0 * D;
    const T *table = rpb ? rpb + ((size_t)(st.plane % g.heads) * NB + (sy - st.y + K - 1)) * NB : nullptr;
    const int tx = sx - qx + K - 1;
    float m = -INFINITY, l = 0.f;
    A acc;
    acc.clear();
    for (int a = st.part; a < K; a += SPLIT) {
        const int row = (sy + a) * W;
        for (int b0 = 0; b0 < nblk; b0 += NBX) {
            float s[NBX][4];
            float gm = -INFINITY;
#pragma unroll
            for (int b = 0; b < NBX; ++b) {
                const int k0 = kx0 + 16 * (b0 + b), kl = k0 + j < W ? k0 + j : W - 1;
                ChannelOp<T, D> ko;
                ko.load(kp + (size_t)(row + kl) * D, grp);
                const f32x4 t = dot_block<T, D>(ko, qo);
                const int c0 = k0 + 4 * grp - sx;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float x = scale * t[r];
                    if (table) x += to_f32(table[a * NB + tx + clamp_to(c0 + r, K - 1)]);
                    s[b][r] = (unsigned)(c0 + r) < (unsigned)K ? x : -INFINITY;
                    gm = fmaxf(gm, s[b][r]);
                }
            }
            gm = fmaxf(gm, __shfl_xor(gm, 16));
            gm = fmaxf(gm, __shfl_xor(gm, 32));
            const float mnew = fmaxf(m, gm), base = mnew == -INFINITY ? 0.f : mnew;   // nothing in reach yet: weights 0
            const float corr = __expf(m - base);
            m = mnew;
            l *= corr;
#pragma unroll
            for (int i = 0; i < A::NB; ++i) acc.acc[i] *= corr;
#pragma unroll
            for (int b = 0; b < NBX; ++b) {
                T wt[NW][4];
                int off[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float p = kWeightUp<T> * __expf(s[b][r] - base);
                    l += p;
                    wt[0][r] = from_f32<T>(p);
                    if constexpr (NW == 2) wt[NW - 1][r] = from_f32<T>(p - to_f32(wt[0][r]));
                    const int kx = kx0 + 16 * (b0 + b) + 4 * grp + r;
                    off[r] = (row + (kx < W ? kx : W - 1)) * D;
                }
                acc.template add<NW>(vp, off, j, wt);
            }
        }
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (grp == 0) {
        wm[st.wave][j] = m;
        wl[st.wave][j] = l;
    }
    acc.to_lds(part[st.wave], j, grp);
    join_waves<SPLIT>();
    const int w0 = st.wave - st.part;   // the strip's first wave
    // the waves' parts of output i: maximum, weighted sum and sum of the weights
    const auto joined = [&](int i, float &mm, float &num, float &den) {
        const int p = i / D, d = i % D;
        mm = wm[w0][p];
#pragma unroll
        for (int t = 1; t < SPLIT; ++t) mm = fmaxf(mm, wm[w0 + t][p]);
        num = den = 0.f;
#pragma unroll
        for (int t = w0; t < w0 + SPLIT; ++t) {
            const float f = wm[t][p] == -INFINITY ? 0.f : __expf(wm[t][p] - mm);   // a wave without rows adds nothing
            num = __builtin_fmaf(f, part[t][p * A::kPitch + d], num);
            den = __builtin_fmaf(f, wl[t][p], den);
        }
        if (den == 0.f) den = NAN;   // every logit -inf
    };
    // (where the sum of the weights is NaN the output is, whatever the weighted sum is)
    const auto spoilt = [](float num, float den) { return den == den && !(fabsf(num) < INFINITY); };
    bool again = false;
    for (int i = st.part * kWave + lane; i < kStrip * D; i += SPLIT * kWave) {
        const int d = i % D, x = st.x0 + i / D;
        if (x >= W) break;   // (the position grows with i)
        float mm, num, den;
        joined(i, mm, num, den);
        again |= spoilt(num, den);
        const size_t n = plane0 + (size_t)st.y * W + x;
        out[n * D + d] = from_f32<T>(num * (1.f / den));
        if (lse != nullptr && d == 0) lse[n] = mm + __logf(den * (1.f / kWeightUp<T>));
    }
    if (__ballot(again) == 0) return;
    // outputs that are not finite once more from their own windows only, a position at a time
    static_assert(kStrip * D % (SPLIT * kWave) == 0);   // (all lanes of a wave stay together)
#pragma unroll 1
    for (int i = st.part * kWave + lane; i < kStrip * D; i += SPLIT * kWave) {
        const int p = i / D, d = i % D;
        float mm, num, den;
        joined(i, mm, num, den);
        const bool redo = st.x0 + p < W && spoilt(num, den);
        for (unsigned long long left = __ballot(redo); left != 0;) {
            const int first = __builtin_ctzll(left), pp = __builtin_amdgcn_readlane(p, first), px = st.x0 + pp, osx = win_start(px, W, K);
            const float mp = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mm), first));
            const size_t n = plane0 + (size_t)st.y * W + px;
            const bool here = redo && p == pp;
            const float own = fused_position<T, D>(q + n * D, kp, vp, table ? table + osx - px + K - 1 : nullptr, scale, mp, W, K, sy, osx, d, here);
            if (here) out[n * D + d] = from_f32<T>(kWeightUp<T> * own * (1.f / den));
            left &= ~__ballot(here);
        }
    }
}

// Logits and fused forward: four waves to a strip while that is what fills the chip; with enough strips each wave keeps
// one to itself, the four of a workgroup one below the other: they read nearly the same rows at the same time, and
// nothing has to be joined.  The weighted sums gain nothing from it (D = 64, k = 9: 198 / 196 us at 21k strips).
// Measured on 14 x 14, 28 x 28, 33 x 70 and 56 x 56 maps, fp32, and f16 where it comes here, time with one wave over time with
// four.  Logits, k = 3 (three rows leave one of four waves idle) and 5: D = 128 at 1.8k strips 0.80 .. 0.91, D = 64 0.96 .. 1.10, narrower 0.96 .. 1.18; all of
// them 0.77 .. 1.10 at 4k, 0.71 .. 0.92 at 40k.  Beyond k = 5, D = 64 and 128 to k = 13: 1.02 .. 1.22 at 3k, 0.87 .. 1.08 at 6k, 0.88 .. 1.06 at 12k;
// narrower heads and wider windows 0.84 .. 1.39, 0.94 .. 1.18, 0.97 .. 1.17, and 0.90 .. 1.19 at 40k: four waves throughout.
int logits_split(const Problem &p) {
    const long long least = p.K <= 5 ? (p.D == 128 ? 1536 : 3584) : p.D >= 64 && p.K <= 13 ? 6144 : LLONG_MAX;   // strips from which on a wave keeps one
    return p.strips() >= least ? 1 : kStripWaves;
}
// The fused forward, likewise: k >= 11 1.39 at 3k strips, 1.29 at 4k and 6k, 0.93 .. 1.08 at 12k, but with D = 128 1.27, 1.21 and 0.84 .. 1.08.  It only comes here
// where the patches of na2d_patch_fwd.hip do not fit the LDS with the waves that a call needs: head vectors of 256 bytes and more from k = 7 on in
// small calls, and in large ones (64 channels of fp32 and 128 of 16 bit from k = 47 on, 128 of fp32 from k = 29 on); shorter ones from k = 31 on, in small calls only.
template <typename T, int D> constexpr bool kLongVector = D * sizeof(T) >= 256;
template <typename T, int D> bool fused_one_wave(const Problem &p) { return p.strips() >= (D == 128 ? 6144 : 12288); }

SShape strip_shape(const Problem &p, int split) {
    const int strips = (p.W + kStrip - 1) / kStrip, per = kStripWaves / split, rows = (p.H + per - 1) / per;
    return SShape{p.heads, p.H, p.W, p.K, strips, rows, p.planes() * rows * strips};
}

}  // namespace

#define NA2D_STRIP_LAUNCH(kern, ...) NA2D_STRIP_LAUNCH_ROWS(1, kern, __VA_ARGS__)
// a grid of `ngroups` workgroups per strip, each with its part of the window rows
#define NA2D_STRIP_LAUNCH_ROWS(ngroups, kern, ...)                                                                        \
    do {                                                                                                                  \
        hipLaunchKernelGGL(kern, dim3(xcd_padded_grid(g.ntiles), ngroups), dim3(kStripThreads), 0, s, __VA_ARGS__, g);   \
        return hipGetLastError();                                                                                         \
    } while (0)
// BODY with T, D and SPLIT bound
#define NA2D_STRIP_DISPATCH(split, ...)                                                                            \
    do {                                                                                                          \
        const SShape g = strip_shape(p, split);                                                                   \
        if (split == 1) { constexpr int SPLIT = 1; NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, __VA_ARGS__)); } \
        else { constexpr int SPLIT = kStripWaves; NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, __VA_ARGS__)); }  \
    } while (0)

// Workgroups per strip for the logits, whose window rows need no joining: one window row to a wave at least, and no more
// than 2048 workgroups (fp32: 1024).  A small call is bound by the chain of loads and stores along a wave's rows (us, one
// group / at most 512 / 1024 / 2048 workgroups, measured while the bias entries were still loaded behind the stores: bf16, D = 16,
// k = 17, 2 x 33 x 17 8.6 / 5.2 / 4.4 / 4.4, 10 x 33 x 17 11.5 / 11.5 / 11.6 / 7.6; fp32, D = 128, k = 5, 16 x 28 x 28 16.4 / 16.4 / 16.5 / 17.6).
static int qk_row_groups(const Problem &p, int ntiles) {
    const int most = (p.K + kStripWaves - 1) / kStripWaves, fill = 4096 / p.elem_bytes() / ntiles;
    return fill < 1 ? 1 : fill < most ? fill : most;
}
hipError_t launch_qk_strip(const Problem &p, const void *x, const void *y, const void *rpb, float scale, void *logits, hipStream_t s) {
    const int split = logits_split(p);
    NA2D_STRIP_DISPATCH(split, NA2D_STRIP_LAUNCH_ROWS(qk_row_groups(p, g.ntiles), (qk_strip_kernel<T, D, SPLIT>), static_cast<const T *>(x),
                                               static_cast<const T *>(y), static_cast<const T *>(rpb), scale, static_cast<T *>(logits)));
    return hipErrorInvalidValue;
}

template <typename T, int D, bool INV>
static hipError_t launch_sum_strip_t(const Problem &p, const T *w, const T *y, float scale, T *out, hipStream_t s) {
    // A launch holds fewer than 2^32 threads; beyond, the runtime takes the number modulo 2^32 and reports nothing.  With a
    // workgroup to a strip, 50 million positions on maps of three columns are more than that (fp32, D = 32, k = 3), so the planes
    // go in as many launches as it takes: one in any other call.  (Logits and fused forward stay below 0.4 of the limit for every
    // problem that comes here: what they store is wider, or a wave keeps a strip to itself.)
    constexpr int kMost = (int)((1ll << 32) / kStripThreads) - 2 * kNumXcd;
    SShape g = strip_shape(p, kStripWaves);
    const int planes = p.planes(), per_plane = g.ntiles / planes, step = kMost / per_plane;
    if (step < 1) return hipErrorInvalidConfiguration;   // (a plane below 2^31 bytes of fp32 has at most 11.2 million strips)
    for (int first = 0; first < planes; first += step) {
        g.ntiles = (planes - first < step ? planes - first : step) * per_plane;
        const size_t q0 = (size_t)first * p.H * p.W;
        hipLaunchKernelGGL((sum_strip_kernel<T, D, INV, kStripWaves>), dim3(xcd_padded_grid(g.ntiles)), dim3(kStripThreads), 0, s,
                           w + q0 * p.K * p.K, y + q0 * D, scale, out + q0 * D, g);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <bool INV>
static hipError_t launch_sum_strip(const Problem &p, const void *w, const void *y, float scale, void *out, hipStream_t s) {
    NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, return (launch_sum_strip_t<T, D, INV>(p, static_cast<const T *>(w),
                                          static_cast<const T *>(y), scale, static_cast<T *>(out), s))));
    return hipErrorInvalidValue;
}
hipError_t launch_av_strip(const Problem &p, const void *w, const void *y, float scale, void *out, hipStream_t s) {
    return launch_sum_strip<false>(p, w, y, scale, out, s);
}
hipError_t launch_inverse_strip(const Problem &p, const void *w, const void *x, float scale, void *out, hipStream_t s) {
    return launch_sum_strip<true>(p, w, x, scale, out, s);
}

// NBX blocks of keys at a time: two while the strip's windows then fit one pass (K <= 17), three for wider ones
template <typename T, int D, int NBX, int SPLIT>
static hipError_t launch_fused_strip_t(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale,
                                       void *out, float *lse, hipStream_t s) {
    const SShape g = strip_shape(p, SPLIT);
    NA2D_STRIP_LAUNCH((fused_strip_kernel<T, D, NBX, SPLIT>), static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                      static_cast<const T *>(rpb), scale, static_cast<T *>(out), lse);
}
hipError_t launch_fused_strip(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale,
                              void *out, float *lse, hipStream_t s) {
    NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, {
        if constexpr (kLongVector<T, D>) {
            if (p.K <= 17) return (launch_fused_strip_t<T, D, 2, kStripWaves>(p, q, k, v, rpb, scale, out, lse, s));
            if (fused_one_wave<T, D>(p)) return (launch_fused_strip_t<T, D, 3, 1>(p, q, k, v, rpb, scale, out, lse, s));
        }
        return (launch_fused_strip_t<T, D, 3, kStripWaves>(p, q, k, v, rpb, scale, out, lse, s));
    }));
    return hipErrorInvalidValue;
}

}  // namespace na2d
