// Fused forward of neighbourhood attention over 4 x 4 query patches for any window side, head dim and storage type (arXiv
// 2204.07143, Eq. 2-4): softmax(scale q K + bias) V of each query's window in one pass over its keys.
//
// A wave keeps a patch of 16 queries and walks its windows' rows of 4 x 4 key blocks; keys and values pass through LDS four map rows at
// a time (na2d_patch.hpp).  The weights leave the matrix cores in the layout in which they enter them again.  Their base is a running
// maximum that is only moved when a logit exceeds it by kSlack: in most blocks no lane has to know another's.  In small calls
// 2, 4 or 8 waves share a patch, a row of blocks each, and are joined in wave order.
//
// In 16 bit a weight enters as a high and a low half, p = hi + lo to 2^-17 of p in bf16.  In fp16 weights are scaled by 2^15 (kUp;
// their sum likewise): 65000 at most, to 2^-22 of themselves down to 2^-18 of the largest and to 2^-40 of the largest below.
//
// A masked product is 0 * v: outputs that are not finite are worked out once more from their own window only.
//
// Measured against the strips of na2d_strip.hip (us, they / this): 64 x 2 x 56 x 56 queries, fp32, 32 channels, k = 7 231 / 119; 4 x 2 x 64 x 64, bf16, 32
// channels, k = 21 45 / 17; 31 maps of 56 x 56, fp16, 128 channels, k = 9 128 / 63.  Per 16 x 16 products 45 vector instructions (the strips 188), and 4 x 4 blocks
// have half the masked products at k = 21.  fp32 is bound by its matrix instructions (512 cycles per block and SIMD: 47 us at the first shape).
#include <limits.h>

#include "na2d_kernels.hpp"
#include "na2d_patch.hpp"

namespace na2d {

namespace {

// waves per SIMD the kernel is built for: two workgroups per compute unit where 128 registers hold a wave
template <typename T, int D> constexpr int kFwdOcc = D * sizeof(T) <= 128 ? 4 : 2;
template <typename T, int D> constexpr int kFwdAtOnce = D * sizeof(T) <= 64 || kFwdOcc<T, D> == 2 ? 2 : 1;
template <typename T> constexpr float kUp = 0.f;          // log2 of what the weights are scaled by
template <> constexpr float kUp<f16_t> = 15.f;
template <typename T> constexpr float kSlack = 20.f;      // by how much (log2) a logit may exceed the base
template <> constexpr float kSlack<f16_t> = 0.98f;        // (2^15.98 is the last that fp16 holds with room for the roundings)

// The outputs and the log-sum-exp of one query from its own window, in raster order: the largest logit, then 64 slots' weights at a time (a
// slot to a lane), then each lane adds up its channels.  A logit that is NaN or +inf makes every output NaN, and once every sum is NaN
// nothing changes any more: where a whole tensor is NaN a few loads are all.
template <typename T, int D>
__device__ __forceinline__ void output_once_more(const T *q, const T *kp, const T *vp, const T *bt, const PatchShape &g, float scale, int iy, int ix,
                                                 T *out, float *lse) {
    constexpr int NU = (D + kWave - 1) / kWave, kChunk = 8;
    const int lane = threadIdx.x % kWave, K = g.K, KK = K * K, W = g.W, sy = win_start(iy, g.H, K), sx = win_start(ix, W, K);
    const T *qi = q + ((size_t)iy * W + ix) * D;
    const auto logit = [&](int first) {   // in units of log2
        const int slot = first + lane < KK ? first + lane : KK - 1, a = slot / K, c = slot - a * K;
        float s = scale * dot_memory<T, D>(qi, kp + ((size_t)(sy + a) * W + sx + c) * D);
        if (bt) s += to_f32(bt[(sy + a - iy + K - 1) * (2 * K - 1) + sx + c - ix + K - 1]);
        return s * kLog2e;
    };
    float m = -INFINITY, l = 0.f;
    bool open = true;
    for (int first = 0; first < KK && open; first += kWave) {
        const float s = logit(first);
        m = fmaxf(m, s);
        open = __ballot(!(s < INFINITY)) == 0;
    }
    if (!open) l = NAN;
#pragma unroll
    for (int x = 1; x < kWave; x *= 2) m = fmaxf(m, __shfl_xor(m, x));
    const float base = m == -INFINITY ? 0.f : m;
    float acc[NU] = {};
    RasterWalk at;
    for (int first = 0; first < KK && !(l != l); first += kWave) {
        float w = __builtin_amdgcn_exp2f(logit(first) - base);
        if (first + lane >= KK) w = 0.f;
        l += w;
        const int n = KK - first < kWave ? KK - first : kWave;
        for (int t0 = 0; t0 < n && open; t0 += kChunk) {
            float wt[kChunk], y[kChunk][NU];
#pragma unroll
            for (int e = 0; e < kChunk; ++e) {   // (their loads do not wait for each other; past the end: once more, not added)
                wt[e] = lane_value(w, (t0 + e) % kWave);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int d = u * kWave + lane < D ? u * kWave + lane : D - 1;
                    y[e][u] = to_f32(vp[((size_t)(sy + at.row) * W + sx + at.col) * D + d]);
                }
                at.next(K, K);
            }
            bool any = false;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
#pragma unroll
                for (int e = 0; e < kChunk; ++e)
                    if (t0 + e < n) acc[u] = __builtin_fmaf(wt[e], y[e][u], acc[u]);
                any |= acc[u] == acc[u];
            }
            open = __ballot(any) != 0;
        }
    }
#pragma unroll
    for (int x = 1; x < kWave; x *= 2) l += __shfl_xor(l, x);
    if (l == 0.f) l = NAN;   // every logit -inf
    const float inv = 1.f / l;
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (u * kWave + lane < D) replace_not_finite(out + ((size_t)iy * W + ix) * D + u * kWave + lane, acc[u] * inv);
    if (lse != nullptr && lane == 0) replace_not_finite(lse + (size_t)iy * W + ix, (base + __builtin_amdgcn_logf(l)) * 0.6931471805599453f);
}

template <typename T, int D>
__global__ __launch_bounds__(kPatchThreads, (kFwdOcc<T, D>)) void patch_fwd_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale, T *__restrict__ out,
    float *__restrict__ lse, PatchShape g) {
    using CV = ChanVec<T, D>;
    using Op = PosOp<T, D>;
    using Sum = PosSum<T, D>;
    constexpr int POSB = Op::POSB, kAtOnce = kFwdAtOnce<T, D>;
    extern __shared__ __align__(16) char lds[];
    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= g.units * g.splits) return;
    const WorkItem work = decode_work(wg, g.heads, g.tiles_y, g.splits, g.gd);
    const int head = work.head, K = g.K, H = g.H, W = g.W, NB = 2 * K - 1, pitch = bias_pitch(K);
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int j = lane & 15, gr = lane >> 4;
    const int lgs = g.lg_split, lg = g.lg_cols, step = 4 << lgs;   // map rows per step
    const int part = wave & ((1 << lgs) - 1), pw = wave >> lgs;    // the wave's row of blocks in a step, and its patch of the tile
    const int bias0 = dynamic_lds(lds), img0 = bias0 + bias_rows(K, g.with_bias) * pitch * 4;
    const int img_bytes = step * g.rw * POSB, stage_bytes = 2 * img_bytes;

    const int tw = 4 << lg, th = (32 >> lgs) >> lg, ty0 = work.ty * th, tx0 = work.tx * tw;
    const int ty1 = ty0 + th - 1 < H - 1 ? ty0 + th - 1 : H - 1;
    const int ry0 = win_start(ty0, H, K), cx0 = win_start(tx0, W, K);   // first key row and column of the tile
    const int nsteps = (win_start(ty1, H, K) + K - ry0 + step - 1) >> (2 + lgs);
    const int sy0 = ty0 + 4 * (pw >> lg), px0 = tx0 + 4 * (lg == 2 && lgs == 0 ? patch_of_wave(pw) : pw & ((1 << lg) - 1));   // this wave's patch
    const bool active = sy0 < H && px0 < W;
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1, px3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1;
    const int pyc = sy0 < H ? sy0 : H - 1, pxc = px0 < W ? px0 : W - 1;
    const int b_lo = (win_start(pyc, H, K) - ry0) >> 2, b_hi = (win_start(sy3, H, K) + K - 1 - ry0) >> 2;   // rows of blocks
    const int ox = win_start(pxc, W, K), nbx = (win_start(px3, W, K) + K - ox + 3) >> 2;
    const int clear_lo = win_start(px3, W, K) - ox;   // columns [clear_lo, K) are in the window of every query of the patch
    const int qy = sy0 + (j >> 2), qx = px0 + (j & 3);
    const bool q_ok = qy < H && qx < W;
    const int iy = qy < H ? qy : H - 1, ix = qx < W ? qx : W - 1;
    const int wy = win_start(iy, H, K), wx = win_start(ix, W, K) - ox;
    const int aoff = ((4 * part + (j >> 2)) * g.rw + (ox - cx0) + (j & 3)) * POSB + gr * CV::kLaneBytes;
    const int toff = Op::lane_offset(lane, g.rw) + (4 * part * g.rw + ox - cx0) * POSB;
    const int u0 = ry0 + gr - iy + K - 1, boff = bias0 + (ox - ix + K - 1 + kBiasPad) * 4;
    const int no_row = boff + (bias_rows(K, g.with_bias) - 1) * pitch * 4;
    const size_t plane_px = (size_t)H * W;
    const int qlin = iy * W + ix;
    const float scale2 = scale * kLog2e, scale2_low = __builtin_fmaf(scale, kLog2e, -scale2) + scale * kLog2eLow;

    auto issue = [&](int b, int s, int par) {
        const size_t off = ((size_t)b * g.heads + head) * plane_px * POSB;
        issue_rows<POSB>(reinterpret_cast<const char *>(k) + off, reinterpret_cast<const char *>(v) + off, H, W, ry0 + step * s, cx0, g.rw,
                         img0 + par * stage_bytes, img_bytes, wave, lane, step);
    };
    if (work.b_begin < work.b_end) issue(work.b_begin, 0, 0);
    stage_bias<T>(g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, K, g.by_pitch, bias0, tid);

    int par = 0;
    for (int b = work.b_begin; b < work.b_end; ++b) {
        const size_t plane = (size_t)b * g.heads + head, plane_off = plane * plane_px * POSB;
        CV qo;
        qo.load(reinterpret_cast<const char *>(q) + plane_off + (unsigned)(qlin * POSB + gr * CV::kLaneBytes));
        settle(qo);
        Sum acc, row;   // (fp32: of a row of blocks, then of the rows: one chain of K * K additions is off by more)
        acc.clear();
        if constexpr (sizeof(T) == 4) row.clear();
        float m = -INFINITY, base = -kUp<T>, l = 0.f;   // running maximum, what the exponents are relative to, the lane's sum of the weights
        // N blocks of a row of blocks, from block column bx on
        auto blocks = [&](auto n, int img, int brow, int bx) {
            constexpr int N = decltype(n)::value;
            const int ka0 = img + aoff + bx * 4 * POSB, vt0 = img + img_bytes + toff + bx * 4 * POSB, b0 = brow + bx * 16;
            CV ka[N];
            f32x4 t[N];
            float bias[N][4];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                ka[i].load_lds(ka0 + i * 4 * POSB);
#pragma unroll
                for (int r = 0; r < 4; ++r) bias[i][r] = *lds_ptr<float>(b0 + i * 16 + r * 4);
                // columns outside the window: weight 0 (before the products: no branch may come between one and its use)
                if (4 * (bx + i) < clear_lo || 4 * (bx + i) + 4 > K) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) bias[i][r] = (unsigned)(4 * (bx + i) + r - wx) < (unsigned)K ? bias[i][r] : -INFINITY;
                }
            }
            float most = -INFINITY;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const f32x4 s = chan_dot<T, D>(ka[i], qo);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (sizeof(T) == 4) t[i][r] = exponent_fp32(s[r], scale2, scale2_low, bias[i][r]);
                    else t[i][r] = __builtin_fmaf(scale2, s[r], bias[i][r]);
                    most = fmaxf(most, t[i][r]);
                }
            }
            Op vt[N];
#pragma unroll
            for (int i = 0; i < N; ++i) vt[i].load_lds(vt0 + i * 4 * POSB);
            if (__ballot(most > m + kSlack<T>)) {
                most = fmaxf(most, __shfl_xor(most, 16));
                most = fmaxf(most, __shfl_xor(most, 32));
                const float mnew = fmaxf(m, most), to = (mnew == -INFINITY ? 0.f : mnew) - kUp<T>;   // nothing in reach yet: weights 0
                const float corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(base - to);
                m = mnew;
                base = to;
                l *= corr;
#pragma unroll
                for (int i = 0; i < Op::NA; ++i) acc.acc[i] *= corr;
                if constexpr (sizeof(T) == 4) {
#pragma unroll
                    for (int i = 0; i < Op::NA; ++i) row.acc[i] *= corr;
                }
            }
            Weights4<T> hi[N], lo[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float p[4], rest[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[r] = __builtin_amdgcn_exp2f(t[i][r] - base);
                    l += p[r];
                    if constexpr (sizeof(T) == 2) rest[r] = p[r] - to_f32(from_f32<T>(p[r]));
                }
                hi[i] = Weights4<T>(p);
                if constexpr (sizeof(T) == 2) lo[i] = Weights4<T>(rest);
            }
            auto &to = sizeof(T) == 4 ? row : acc;
            if constexpr (N == 2) to.add2(vt[0], hi[0], vt[1], hi[1]);
            else if constexpr (kAtOnce == 2) to.add_last(vt[0], hi[0]);
            else to.add(vt[0], hi[0]);
            if constexpr (sizeof(T) == 2) {
                if constexpr (N == 2) to.add2(vt[0], lo[0], vt[1], lo[1]);
                else if constexpr (kAtOnce == 2) to.add_last(vt[0], lo[0]);
                else to.add(vt[0], lo[0]);
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
            const int br = (s << lgs) + part;   // this wave's row of blocks
            if (active && br >= b_lo && br <= b_hi) {
                const int u = u0 + 4 * br, uc = u < 0 ? 0 : (u < NB - 1 ? u : NB - 1);
                const bool rowok = (unsigned)(ry0 + 4 * br + gr - wy) < (unsigned)K;
                const int brow = rowok ? boff + (g.with_bias ? uc * pitch * 4 : 0) : no_row;
                int bx = 0;
                for (; bx + kAtOnce <= nbx; bx += kAtOnce) blocks(IntC<kAtOnce>{}, img, brow, bx);
                if (kAtOnce > 1 && bx < nbx) blocks(IntC<1>{}, img, brow, bx);
                if constexpr (sizeof(T) == 4) acc.take(row);
            }
            if (g.nstage == 1 && (!last || b + 1 < work.b_end)) {
                workgroup_sync();   // nobody still reads the rows
                issue(last ? b + 1 : b, last ? 0 : s + 1, 0);
            }
        }
        if constexpr (sizeof(T) == 2) acc.settle();
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (lgs > 0) {
            // the waves of a patch, joined in wave order by the first (one tile per workgroup: the images are free)
            workgroup_sync();
            constexpr int kPart = Op::NA * 1024 + 512;   // sums, then base and l, of a wave
            const int mine = img0 + wave * kPart;
            if (part > 0) {
#pragma unroll
                for (int i = 0; i < Op::NA; ++i) *lds_ptr<f32x4>(mine + i * 1024 + lane * 16) = acc.acc[i];
                *lds_ptr<f32x2>(mine + Op::NA * 1024 + lane * 8) = f32x2{m == -INFINITY ? -INFINITY : base, l};
            }
            workgroup_sync();
            if (part > 0) return;
            for (int o = 1; o < (1 << lgs); ++o) {
                const int from = img0 + (wave + o) * kPart;
                const f32x2 other = *lds_ptr<f32x2>(from + Op::NA * 1024 + lane * 8);
                if (m == -INFINITY) base = other.x == -INFINITY ? base : other.x;
                const float to = fmaxf(base, other.x);
                const float ca = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(base - to), cb = other.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(other.x - to);
                if (other.x > -INFINITY && m == -INFINITY) m = 0.f;   // (from here on only: something has been in reach)
                base = to;
                l = __builtin_fmaf(other.y, cb, l * ca);
#pragma unroll
                for (int i = 0; i < Op::NA; ++i) {
                    const f32x4 x = *lds_ptr<f32x4>(from + i * 1024 + lane * 16);
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc.acc[i][r] = __builtin_fmaf(x[r], cb, acc.acc[i][r] * ca);
                }
            }
        }
        if (!active) continue;
        if (l == 0.f) l = NAN;   // every logit -inf
        const float inv = 1.f / l;
        if (q_ok) {
            acc.store(reinterpret_cast<char *>(out) + plane_off, (unsigned)(qlin * POSB), gr, inv);
            if (lse != nullptr && gr == 0) (lse + plane * plane_px)[(unsigned)qlin] = (base + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
        }
        // (a sum of the weights that is NaN may be so for a key outside of the window: the logit itself is not finite there)
        const float odd = acc.not_finite() + l;
        const unsigned long long again = __ballot(odd != odd);
        if (again) {
            wait_global_loads();   // (the stores above come first)
            PatchShape gc = g;     // (nothing of this is prepared outside of the branch)
            asm volatile("" : "+s"(gc.H), "+s"(gc.W), "+s"(gc.K));
            for (unsigned cols = (unsigned)((again | (again >> 16) | (again >> 32) | (again >> 48)) & 0xffffu); cols; cols &= cols - 1) {
                const int c = __builtin_ctz(cols), cy = sy0 + (c >> 2), cx = px0 + (c & 3);
                if (cy < H && cx < W)
                    output_once_more<T, D>(q + plane * plane_px * D, k + plane * plane_px * D, v + plane * plane_px * D,
                                           g.with_bias ? rpb + (size_t)head * NB * NB : nullptr, gc, scale, cy, cx, out + plane * plane_px * D,
                                           lse ? lse + plane * plane_px : nullptr);
            }
        }
    }
}

struct FwdPlan {
    PatchShape s;
    int lds;
    bool ok, enough_waves;
};
// Waves per patch: as many as fill the chip, and no more than the patch has rows of blocks.  Measured (us with 1 / 2 / 4, fp32 and fp16, 16 to 128
// channels, k = 3 .. 63): 64 patches 20 / 16 / 13 .. 49 / 30 / 29, 162 patches 34 / 21 / 17, 58 / 33 / 34, 800 patches 35 / 23 / 32, 27 / 18 / 27, 14 / 13 / 14, 7000 patches
// 107 / 132 / 176, 37 / 39 / 50 (where one row of blocks is all there is to a step, more waves only wait).
int waves_per_patch(long long patches, int block_rows) {
    const int most = patches <= 200 ? 3 : patches <= 400 ? 2 : patches <= 2000 ? 1 : 0;
    int lgs = 0;
    while (lgs < most && (1 << lgs) < block_rows) ++lgs;
    return lgs;
}
// A plan with as many waves per patch as wanted, or with fewer where the LDS does not hold a step of all of them.
FwdPlan fwd_plan(const Problem &p, bool bias) {
    FwdPlan pl{};
    const int K = p.K, posb = p.D * p.elem_bytes(), pitch = bias_pitch(K), table = bias_rows(K, bias) * pitch * 4;
    const long long patches = (long long)p.planes() * ((p.H + 3) / 4) * ((p.W + 3) / 4);
    const int want = waves_per_patch(patches, (K + 6) / 4);
    for (int lgs = want; lgs >= 0 && !pl.ok; --lgs) {
        const int step = 4 << lgs;
        // the tile's shape: the one that takes the fewest steps of streamed rows
        long long least = LLONG_MAX;
        for (int lg = 3 - lgs; lg >= 0; --lg) {
            const int tw = 4 << lg, th = (32 >> lgs) >> lg, rows = th + K - 1 < p.H ? th + K - 1 : p.H;
            if (th > 16) continue;
            const int rw = image_row(p.W, K, tw, posb, [&](int x) { return win_start(x, p.W, K); }, [&](int x) { return win_start(x, p.W, K) + K - 1; });
            int lds;
            int n = image_buffers(table, 2 * step * rw * posb, lds);
            if (n == 2 && lgs > 0 && rows <= step) n = 1, lds = table + 2 * step * rw * posb;   // one step, one tile: nothing to load ahead
            const int joined = table + 8 * (p.D / 16 * 1024 + 512);                            // (what joining the waves of a patch takes)
            if (n == 0 || (lgs > 0 && joined > 160 * 1024)) continue;
            if (lgs > 0 && lds < joined) lds = joined;
            const int tiles_x = (p.W + tw - 1) / tw, tiles_y = (p.H + th - 1) / th;
            const long long steps = (long long)tiles_x * tiles_y * ((rows + step - 1) / step);
            if (steps >= least) continue;
            least = steps;
            UnitSplit us;
            us.units = tiles_x * tiles_y * p.heads;
            us.splits = lgs > 0 ? p.B : 2048 / us.units;   // (the waves of a patch are joined in the images: one tile per workgroup)
            us.splits = us.splits < 1 ? 1 : us.splits < p.B ? us.splits : p.B;
            us.gd = make_grid_decode(tiles_x, tiles_y, p.heads, p.B, us.splits);
            pl.s = PatchShape{p.H, p.W, K, p.heads, tiles_y, us.units, us.splits, rw, lgs, lg, n, 1, bias ? 1 : 0, 0, us.gd, make_fastdiv(pitch)};
            pl.lds = lds;
            pl.ok = true;
            pl.enough_waves = lgs >= (want < 2 ? want : 2);
        }
    }
    return pl;
}

}  // namespace

// Where the patches are faster than strips (na2d_strip.hip): wherever the LDS holds what the call's size asks for.  Time over that of the strips
// (14 x 14 to 70 x 70 maps, 800 to 100k queries): fp32 0.45 .. 0.85 from 12000 queries on, 0.9 .. 1.1 below (launch); fp16, k >= 15 and
// 128 channels from k = 9 on, 0.31 .. 0.9.  With fewer waves per patch than wanted 1.04 .. 2.7 (fp32, 64 channels, k = 31, one 33 x 70 map 37 -> 101).
bool patch_fwd_preferred(const Problem &p) {
    const FwdPlan pl = fwd_plan(p, true);
    return pl.ok && pl.enough_waves;
}

hipError_t launch_patch_fwd(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale, void *out, float *lse, hipStream_t s) {
    const FwdPlan pl = fwd_plan(p, rpb != nullptr);
    if (!pl.ok) return hipErrorInvalidValue;
    NA2D_DISPATCH_T(p.dtype, NA2D_DISPATCH_D(p.D, {
        static LdsAllowed allowed;
        if (hipError_t e = allow_lds(patch_fwd_kernel<T, D>, 160 * 1024, allowed); e != hipSuccess) return e;
        hipLaunchKernelGGL((patch_fwd_kernel<T, D>), dim3(xcd_padded_grid(pl.s.units * pl.s.splits)), dim3(kPatchThreads), pl.lds, s,
                           static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v), static_cast<const T *>(rpb), scale,
                           static_cast<T *>(out), lse, pl.s);
        return hipGetLastError();
    }));
    return hipErrorInvalidValue;
}

}  // namespace na2d
