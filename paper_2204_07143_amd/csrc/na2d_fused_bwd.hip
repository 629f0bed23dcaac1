// Fused neighbourhood attention backward on the matrix cores (f16 / bf16, K <= 9): the gradients
// of q, k, v and of the bias table from q, k, v, dout and the log-sum-exp of every query that the
// fused forward left behind; the k*k attention weights and their gradients never reach memory
// (arXiv 2204.07143: Eq. 2-4 differentiated; Appendix A lists the five gradients).
//
//   P[i, j]  = exp(scale <q_i, k_j> + B(i, j) - lse_i)           recomputed per tile
//   dP[i, j] = <dout_i, v_j>
//   delta_i  = sum_j P[i, j] dP[i, j]
//   dS[i, j] = P[i, j] (dP[i, j] - delta_i)
//   dq_i = scale sum_j dS[i, j] k_j      dB = sum over the queries of dS, per relative position
//   dk_j = scale sum_i dS[i, j] q_i      dv_j = sum_i P[i, j] dout_i
//
// Two kernels.  The first keeps 4 x 4 query patches (rows of P: dq, dB, and delta, which it leaves in
// the workspace for the second); the second keeps 4 x 4 key patches (columns of P: dk, dv).
#include "na2d_kernels.hpp"
#include "na2d_mfma.hpp"
#include "na2d_rpb_final.hpp"
#include "na2d_tile.hpp"

namespace na2d {

template <typename T> __device__ __forceinline__ uint32_t pack2_t(float a, float b) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef T tx2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, tx2_t));
}
// ---- part 1: query patches -> dq, delta, partial dB ------------------------------------------
//
// Same decomposition as the fused forward: eight waves share a 16 x 8 query tile, one 4 x 4 patch
// each; a workgroup keeps one tile position and one head and walks a range of the batch, so the
// window mask, the bias table and every address are built once; the key and the value halo of a
// tile reach one of two LDS buffer pairs by direct loads while the previous tile is computed.
// Two sweeps over the 16-position blocks of the patch halo.  The first evaluates
//   S^T = K_blk Q^T, dP^T = V_blk dout^T    (keys / values as 16-byte A operands, q / dout of the lane's
//                                            query as B operand)
// for P, which stays in registers, and delta = sum P dP (a query's positions are spread over 4 lanes: two
// cross-lane steps), the second dP^T once more for
//   dS^T = P (dP - delta)                    in registers, already in the B-operand layout of
//   dq^T += K_blk^T dS^T                     the half-depth MFMA (keys through the transposing LDS read).
// The kernel is bound by vector instructions (75 % of the issue slots at 64 x 2 x 56 x 56, K = 7, f16, with both
// products and the exponential in both sweeps): P costs 3 + 1 of them per result and one register to keep, dP one
// MFMA and one LDS read per 16 x 16 block to evaluate again.  Each block's operands are read from LDS one block
// ahead, and ahead of the table adds, since a wave's LDS operations return in order.  Together with a bound of |dP|
// in one instruction per two results: 54.7 -> 45.4 us there, 36 -> 32 us at bf16 128 x 8 x 14 x 14.
// Every dS is also added to its cell of a (2K-1)^2 table in LDS (Eq. 2's B differentiated: the bias cell of a
// (query, position) pair depends on their offset only).  The tables are 64-bit fixed point with 32 fraction
// bits and the adds are integer atomics: on this chip an LDS integer add costs a few cycles per wave
// instruction where the floating-point add costs about 200, and integer addition does not depend on the
// order of the operands, so the bias gradient is bitwise reproducible although waves share tables.
// A dS is converted in two steps so that its precision follows its size: a lane bounds the dS of its query
// in a plane by B = max |dP| + |delta| (from the first sweep), takes sh = max(0, exponent(B) + 32 - 30), turns
// dS 2^(32 - sh) into a 32-bit integer (below 2^30 in magnitude, truncated: an error below 2^-30 B) and shifts
// it left by sh as a 64-bit integer.  Small gradients therefore keep an absolute resolution of 2^-32 (2.3e-10),
// large ones a relative one of 2^-30, and a workgroup's 64-bit sums (about 2^11 terms per cell) stay exact while
// |dS| < 2^20; beyond that they wrap.  A workgroup's tables, added up and converted to fp32 at the end, are
// one partial bias gradient.  (A NaN dS counts as 0.)
template <typename T, int K>
struct FbwdQCfg {
    using P = Patch<K>;
    static constexpr int STRIPS = 2;
    static constexpr int WAVES = 4 * STRIPS;
    static constexpr int TY = 4 * STRIPS;
    static constexpr int HALO_H = TY + K - 1, HALO_W = kTileX + K - 1;
    using Halo = HaloDma<T, HALO_H, HALO_W, WAVES>;
    static constexpr int NB = 2 * K - 1, CELLS = NB * NB;
    static constexpr int NPAIR = (P::NBLK + 1) / 2;
    static constexpr int NBLK2 = 2 * NPAIR;
    static constexpr int kThreads = kWave * WAVES;
    static constexpr int kHaloBytes = Halo::kBytes;
    static constexpr int kStageBytes = 2 * kHaloBytes;   // keys, then values
    // Two buffer pairs where two workgroups then still share a compute unit's LDS; one pair, reloaded between tiles
    // while the other workgroup computes, where that is what makes them fit (K = 9)
    static constexpr int kTblPad = 3;                    // cells in front of and behind a table (see the cell offsets)
    static constexpr int kTblBytes = (CELLS + 2 * kTblPad) * 8;
    static constexpr bool kOneStage = 2 * kStageBytes + kTblBytes > 80 * 1024;
    static constexpr int NSTAGE = kOneStage ? 1 : 2;
    // Bias-gradient tables behind the buffers, 64-bit fixed point (see above): as many as fit beside two
    // workgroups' buffers in a compute unit's 160 KB, at most one per wave
    static constexpr int kTblFit = (80 * 1024 - NSTAGE * kStageBytes) / kTblBytes;
    static constexpr int NTBL = kTblFit >= WAVES ? WAVES : (kTblFit >= 4 ? 4 : (kTblFit >= 2 ? 2 : 1));
    static_assert(kTblFit >= 1, "no room for a bias-gradient table");
    static constexpr int kFracBits = 32;   // fraction bits of the tables
    static constexpr int kLdsBytes = NSTAGE * kStageBytes + NTBL * kTblBytes;
};

template <typename T, int K, bool RPB>
__global__ __launch_bounds__(512, 4) void fbwd_q_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                        const T *__restrict__ v, const T *__restrict__ rpb, float scale,
                                                        const float *__restrict__ lse, const T *__restrict__ dout,
                                                        T *__restrict__ dq,
                                                        float *__restrict__ stat,
                                                        float *__restrict__ rpb_partial,
                                                        int H, int W, int heads, int nb, int tiles_y, int units, int splits, GridDecode gd,
                                                        int half_dim) {
    using C = FbwdQCfg<T, K>;
    using P = Patch<K>;
    static_assert(C::kThreads == 512, "launch bounds");
    constexpr float kLog2e = 1.4426950408889634f;
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int strip = wave >> 2, p = patch_of_wave(wave);
    const int j = lane & 15, g = lane >> 4, jy = j >> 2, jx = j & 3;
    const int lds0 = lds_addr(lds);

    const int wg = xcd_contiguous_block(blockIdx.x, gridDim.x);
    if (wg >= units * splits) return;
    // neighbouring workgroups take neighbouring tile positions of the same planes (the position index
    // runs fastest), so the positions whose halos overlap run at the same time on the same XCD and
    // the overlap is read from HBM once
    const WorkItem work = decode_work(wg, heads, tiles_y, splits, gd);
    const int head = work.head, ty0 = work.ty * C::TY, tx0 = work.tx * kTileX;
    const int b_begin = work.b_begin, b_end = work.b_end;

    const int hoy = halo_origin(ty0, C::TY, H, K), hox = halo_origin(tx0, kTileX, W, K);   // tile halo origin
    const int sy0 = ty0 + 4 * strip, px0 = tx0 + 4 * p;                                     // this wave's patch
    const bool active = sy0 < H && px0 < W;
    const int oy = halo_origin(sy0 < H ? sy0 : H - 1, 4, H, K), ox = halo_origin(px0 < W ? px0 : W - 1, 4, W, K);
    const int dy = oy - (sy0 - P::R), dx = ox - (px0 - P::R);   // 0 away from the borders
    const int qy = sy0 + jy, qx = px0 + jx;
    const bool q_ok = qy < H && qx < W;

    typename C::Halo halo;
    halo.init(wave, lane);
    int hoff[C::Halo::PER_WAVE];
    // (half_dim: 16-channel heads; see kHalfDimChunks)
    const int pitch = half_dim ? Traits<T>::kKeyBytes / 2 : Traits<T>::kKeyBytes, chunk_mask = half_dim ? kHalfDimChunks : 3;
    halo.offsets(H, W, hoy, hox, hoff, pitch, chunk_mask);
    const int qlin = (qy < H - 1 ? qy : H - 1) * W + (qx < W - 1 ? qx : W - 1);   // this lane's query inside a plane
    const size_t plane_bytes = (size_t)H * W * pitch;
    // per plane: both halos into LDS; this lane's 16 bytes (channels 8g .. 8g + 7) of q and dout of its query
    // and the query's log-sum-exp into registers
    u32x4 qnext, dnext;
    float lnext;
    auto issue = [&](int b, int par) {
        const size_t plane = (size_t)b * heads + head;
        const size_t off = plane * plane_bytes;
        C::Halo::issue_at(reinterpret_cast<const char *>(k) + off, hoff, lds0 + par * C::kStageBytes, wave);
        C::Halo::issue_at(reinterpret_cast<const char *>(v) + off, hoff, lds0 + par * C::kStageBytes + C::kHaloBytes, wave);
        const size_t qo = off + qlin * pitch + (g & chunk_mask) * 16;
        qnext = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(q) + qo);
        dnext = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(dout) + qo);
        lnext = lse[plane * H * W + qlin];
    };
    if (b_begin < b_end) issue(b_begin, 0);

    // Operand addresses inside the first buffer pair; those of the transposing reads are recomputed where they
    // are used, from an opaque copy of the lane index (eight more registers held across the loop cost more
    // than the arithmetic).
    // Keys / values as A operand rows: halo position 16b + j, bytes [16g, 16g+16).  Keys through the
    // transposing read: inside its group of 16 lanes, lane j points at four channels of halo position
    // 16b + 4g + j / 4 and receives the j-th channel of positions 16b + 4g .. + 3; the channels are dealt so
    // that MFMA row m of half hf is channel 8 (m / 4) + 4 hf + m % 4, which leaves a lane with the eight
    // consecutive channels 8g .. 8g + 7 of its query (one 16-byte store).
    const int kbase = lds0 + ((oy - hoy) * C::HALO_W + (ox - hox)) * Traits<T>::kKeyBytes;   // halo position 0 of the patch
    auto row_addr = [&](int lv, int b) {   // A operand row of block b
        int h = 16 * b + (lv & 15);
        h = h < P::NKEY ? h : P::NKEY - 1;   // past the end: any real position (its dS is zero)
        const int hy = P::row_of(h), hx = h - hy * P::PW;
        return kbase + (hy * C::HALO_W + hx) * Traits<T>::kKeyBytes + (lv >> 4) * 16;
    };
    int koff[P::NBLK];   // used twice per plane: kept
#pragma unroll
    for (int b = 0; b < P::NBLK; ++b) koff[b] = row_addr(lane, b);
    auto tr_addr = [&](int lv, int b) {   // transposing read of block b
        int h = 16 * b + 4 * (lv >> 4) + ((lv & 15) >> 2);
        h = h < P::NKEY ? h : P::NKEY - 1;
        const int hy = P::row_of(h), hx = h - hy * P::PW;
        return kbase + (hy * C::HALO_W + hx) * Traits<T>::kKeyBytes + (lv & 3) * 16;
    };
    // bias of (this lane's query, halo position), as stored (see bias_to_f16), -inf outside the query's window,
    // as packed fp16 pairs; cell[] is the position's cell in the bias table (-1 outside the window).  Built per
    // group of four consecutive halo positions: those of them inside the window are in one halo row (a halo row
    // holds K + 3 positions, the window K), normally the row of the first position; when that one is already
    // right of the window the group runs on into the next halo row and only that part can be inside.
    f16x2 biasm[P::NEL / 2];
    auto cell_group = [&](int lv, int G, int (&cell)[4]) {   // lv: the lane index (passed in so that the two uses share nothing)
        const int gg = lv >> 4, yy = (lv & 15) >> 2, xx = lv & 3;
        const int cy = sy0 + yy, cx = px0 + xx;
        const bool ok = cy < H && cx < W;
        const int wy = win_start(cy < H ? cy : H - 1, H, K) - oy, wx = win_start(cx < W ? cx : W - 1, W, K) - ox;
        const int h0 = 16 * G + 4 * gg;
        const int hy0 = P::row_of(h0), hx0 = h0 - hy0 * P::PW;
        const bool wrap = hx0 > wx + K - 1;
        const int hy = hy0 + (wrap ? 1 : 0), hxf = hx0 - (wrap ? P::PW : 0);
        const int a = hy - wy;
        const int c0 = (ok && (unsigned)a < (unsigned)K) ? hxf - wx : 64;   // no row of the window: every column test fails
        const int cell0 = (hy - yy + P::R + dy) * C::NB + (hxf - xx + P::R + dx);
#pragma unroll
        for (int i = 0; i < 4; ++i) cell[i] = (unsigned)(c0 + i) < (unsigned)K ? cell0 + i : -1;
    };
    // Where the results of block G are added: byte offset of the cell of result 4G inside a table; results 4G + 1 .. + 3
    // go to the three cells behind it (the cells of a group that lie inside the window are neighbours in one row of
    // the table).  Results outside the window are exactly 0 and adding them changes nothing, so they may go to any
    // cell: those of a group with a position inside the window simply land next to it, up to three cells in front of
    // or behind the table (kTblPad); a group with no position inside the window gets four cells that differ from lane
    // to lane, so that the adds of one instruction do not pile up on one address.
    int coff[RPB ? P::NBLK : 1];
    {
        const T *tbl = rpb != nullptr ? rpb + (size_t)head * C::CELLS : nullptr;
        constexpr int GB = K > 7 ? 2 : 4;   // groups per batch of bias loads (a batch of temporaries at a time)
#pragma unroll
        for (int G0 = 0; G0 < P::NBLK; G0 += GB) {
            int cell[4 * GB];
            f16_t bias[4 * GB];
#pragma unroll
            for (int u = 0; u < GB; ++u) {
                int c4[4] = {-1, -1, -1, -1};
                if (G0 + u < P::NBLK) cell_group(lane, G0 + u, c4);
#pragma unroll
                for (int i = 0; i < 4; ++i) cell[4 * u + i] = c4[i];
                if constexpr (RPB) {
                    if (G0 + u < P::NBLK) {
                        int first = -1;   // cell of result 4G, worked back from the first one inside the window
#pragma unroll
                        for (int i = 3; i >= 0; --i) first = c4[i] >= 0 ? c4[i] - i : first;
                        const bool any = (c4[0] & c4[1] & c4[2] & c4[3]) >= 0;
                        coff[G0 + u] = ((any ? first : lane % (C::CELLS - 3)) + C::kTblPad) * 8;
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 4 * GB; ++e) bias[e] = (f16_t)0.f;
            if (tbl != nullptr) {
#pragma unroll
                for (int e = 0; e < 4 * GB; ++e) bias[e] = bias_to_f16(tbl[cell[e] < 0 ? 0 : cell[e]]);
            }
#pragma unroll
            for (int e = 0; e < 4 * GB; ++e)
                if (4 * G0 + e < P::NEL) biasm[(4 * G0 + e) >> 1][e & 1] = cell[e] >= 0 ? bias[e] : (f16_t)-INFINITY;
            if constexpr (K > 7) __builtin_amdgcn_sched_barrier(0);
        }
    }
    const int tbl0 = lds0 + C::NSTAGE * C::kStageBytes;
    const int mytbl = tbl0 + (wave % C::NTBL) * C::kTblBytes;
    if constexpr (RPB) {
        for (int i = tid; i < C::NTBL * (C::kTblBytes / 8); i += C::kThreads) *lds_ptr<unsigned long long>(tbl0 + i * 8) = 0ull;
    }

    auto compute = [&](auto par_c, const u32x4 &qreg, const u32x4 &dreg, float lse1, int b) {
        constexpr int PAR = decltype(par_c)::value;
        const float lse2 = lse1 * kLog2e;
        if (!active) return;
        int lv = lane;
        asm volatile("" : "+v"(lv));
        // the packed table stays packed: without this the conversions to fp32 are hoisted out of the loop over
        // the planes and take 28 registers instead of 14
#pragma unroll
        for (int e = 0; e < P::NEL / 2; ++e) asm volatile("" : "+v"(biasm[e]));
        auto key_rows = [&](int bk) { return *lds_ptr<u32x4>(koff[bk] + PAR * C::kStageBytes); };
        auto value_rows = [&](int bk) { return *lds_ptr<u32x4>(koff[bk] + PAR * C::kStageBytes + C::kHaloBytes); };
        auto weight = [&](int e, float sv) {   // P of result e, 0 outside the window (bias -inf)
            return __builtin_amdgcn_exp2f(__builtin_fmaf(__builtin_fmaf(scale, sv, (float)biasm[e >> 1][e & 1]), kLog2e, -lse2));
        };
        // sweep 1: P, delta
        float delta = 0.f, dpmax = 0.f;
        float pw[P::NEL];
        constexpr bool kAhead = K <= 7;   // operands one block ahead: up to 123 of the 128 registers; K = 9 has none to spare
        u32x4 kr, vr;
        if constexpr (kAhead) kr = key_rows(0), vr = value_rows(0);
#pragma unroll
        for (int bk = 0; bk < P::NBLK; ++bk) {
            if constexpr (!kAhead) kr = key_rows(bk), vr = value_rows(bk);
            const f32x4 sacc = mfma_16x16x32<T>(kr, qreg, f32x4{0.f, 0.f, 0.f, 0.f});
            const f32x4 pacc = mfma_16x16x32<T>(vr, dreg, f32x4{0.f, 0.f, 0.f, 0.f});
            if constexpr (kAhead) {
                if (bk + 1 < P::NBLK) kr = key_rows(bk + 1);
                vr = value_rows(bk + 1 < P::NBLK ? bk + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pw[4 * bk + r] = weight(4 * bk + r, sacc[r]);
                delta = __builtin_fmaf(pw[4 * bk + r], pacc[r], delta);
            }
            if constexpr (RPB) {
#pragma unroll
                for (int r = 0; r < 4; ++r) dpmax = __builtin_elementwise_maximum(dpmax, __builtin_fabsf(pacc[r]));
            }
            __builtin_amdgcn_sched_barrier(0);   // keeps the blocks from being evaluated all at once
        }
        delta = column_sum(delta);
        // fixed-point conversion of this lane's dS in this plane: |dS| <= P |dP - delta| <= dpmax + |delta|
        float fx_scale = 0.f;
        int fx_shift = 0;
        if constexpr (RPB) {
            const int ex = __builtin_amdgcn_frexp_expf(dpmax + fabsf(delta));   // bound < 2^ex
            fx_shift = ex + C::kFracBits - 30;
            fx_shift = fx_shift < 0 ? 0 : (fx_shift > 32 ? 32 : fx_shift);
            fx_scale = __builtin_ldexpf(1.f, C::kFracBits - fx_shift);
        }
        // sweep 2: dP again, dS, dq (one block at a time: the half-depth MFMA takes the four positions a lane holds)
        f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int bk = 0; bk < P::NBLK; ++bk) {
            if constexpr (!kAhead) vr = value_rows(bk);
            const f32x4 pacc = mfma_16x16x32<T>(vr, dreg, f32x4{0.f, 0.f, 0.f, 0.f});
            if (kAhead && bk + 1 < P::NBLK) vr = value_rows(bk + 1);
            const int ta = tr_addr(lv, bk) + PAR * C::kStageBytes;
            const u32x2 kt[2] = {lds_read_tr16(ta), lds_read_tr16(ta + 8)};
            __builtin_amdgcn_sched_barrier(0);   // the reads ahead of the adds: a wave's LDS operations return in order
            float dsv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = 4 * bk + r;
                dsv[r] = pw[e] * (pacc[r] - delta);   // exactly 0 outside the window
                if constexpr (RPB) {
                    const long long fx = (long long)(int)(dsv[r] * fx_scale) << fx_shift;   // truncated, saturating; NaN -> 0
                    __hip_atomic_fetch_add(lds_ptr<unsigned long long>(mytbl + coff[bk] + 8 * r),
                                           (unsigned long long)fx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            const uint32_t b0 = pack2_t<T>(dsv[0], dsv[1]), b1 = pack2_t<T>(dsv[2], dsv[3]);
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const u32x2 a2 = kt[hf];
                o[hf] = mfma_16x16x16<T>(a2.x, a2.y, b0, b1, o[hf]);
                if constexpr (Traits<T>::kDtype == NA2D_BF16) {
                    // bf16 keeps 8 significant bits: a second operand carries the rounding remainder of dS so
                    // that the product sees it to 16 bits
                    const uint32_t l0 = pack2_t<T>(dsv[0] - to_f32(from_f32<T>(dsv[0])), dsv[1] - to_f32(from_f32<T>(dsv[1])));
                    const uint32_t l1 = pack2_t<T>(dsv[2] - to_f32(from_f32<T>(dsv[2])), dsv[3] - to_f32(from_f32<T>(dsv[3])));
                    o[hf] = mfma_16x16x16<T>(a2.x, a2.y, l0, l1, o[hf]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (q_ok) {
            const size_t plane = (size_t)b * heads + head;
            char *dst = reinterpret_cast<char *>(dq) + plane * plane_bytes + qlin * pitch + g * 16;
            if (!half_dim || g < 2)
                store16_stream(dst, u32x4{pack2_t<T>(o[0][0] * scale, o[0][1] * scale), pack2_t<T>(o[0][2] * scale, o[0][3] * scale),
                                          pack2_t<T>(o[1][0] * scale, o[1][1] * scale), pack2_t<T>(o[1][2] * scale, o[1][3] * scale)});
            if (g == 0) {   // for the key-patch kernel: the log-sum-exp, natural, and delta
                typedef float f32x2_t __attribute__((ext_vector_type(2)));
                *reinterpret_cast<f32x2_t *>(stat + 2 * (plane * H * W + qlin)) = f32x2_t{lse1, delta};
            }
        }
    };

    int b = b_begin;
    auto step = [&](auto par_c) {
        constexpr int PAR = decltype(par_c)::value;
        wait_global_loads();   // this tile's halos and the lane's query data have landed
        workgroup_sync();       // ... for every wave, and nobody still reads the other buffer pair
        const bool upper = half_dim && g >= 2;   // lanes whose channels a 16-channel head does not have
        const u32x4 qreg = upper ? u32x4{0u, 0u, 0u, 0u} : qnext, dreg = upper ? u32x4{0u, 0u, 0u, 0u} : dnext;
        const float lse1 = lnext;
        if constexpr (C::kOneStage) {
            compute(par_c, qreg, dreg, lse1, b);
            if (b + 1 < b_end) {
                workgroup_sync();   // nobody still reads the halos
                issue(b + 1, 0);
            }
        } else {
            if (b + 1 < b_end) issue(b + 1, PAR ^ 1);
            compute(par_c, qreg, dreg, lse1, b);
        }
        ++b;
    };
    while (b < b_end) {
        step(IntC<0>{});
        if constexpr (!C::kOneStage) {
            if (b < b_end) step(IntC<1>{});
        }
    }

    if constexpr (RPB) {
        // the tables added up (integers: any order), then to fp32: one partial bias gradient per workgroup
        workgroup_sync();
        for (int cell = tid; cell < C::CELLS; cell += C::kThreads) {
            long long sum = 0;
#pragma unroll
            for (int t = 0; t < C::NTBL; ++t) sum += (long long)*lds_ptr<unsigned long long>(tbl0 + t * C::kTblBytes + (cell + C::kTblPad) * 8);
            // row of this workgroup's partial: the partials of a head follow each other (rpb_cell_stride)
            rpb_partial[(size_t)((head * splits + work.split) * gd.npos + work.pos) * rpb_cell_stride(C::CELLS) + cell] =
                (float)((double)sum * (1.0 / 4294967296.0));   // 2^-32
        }
    }
}

template <typename T, int K>
static hipError_t launch_fbwd_q_t(const Problem &p, const void *q, const void *k, const void *v, const void *rpb,
                                  float scale, const float *lse, const void *dout, void *dq, float *stat,
                                  float *rpb_partial, hipStream_t s) {
    using C = FbwdQCfg<T, K>;
    static_assert(C::kLdsBytes <= 80 * 1024, "two workgroups share the LDS of a compute unit");
    const int tiles_x = (p.W + kTileX - 1) / kTileX, tiles_y = (p.H + C::TY - 1) / C::TY;
    const UnitSplit us = unit_split(tiles_x, tiles_y, p.heads, p.B);
    const bool with_rpb = rpb_partial != nullptr;
    auto kern = with_rpb ? fbwd_q_kernel<T, K, true> : fbwd_q_kernel<T, K, false>;
    static LdsAllowed allowed[2];
    if (hipError_t e = allow_lds(kern, C::kLdsBytes, allowed[with_rpb]); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(xcd_padded_grid(us.units * us.splits)), dim3(C::kThreads), C::kLdsBytes, s,
                       static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                       static_cast<const T *>(rpb), scale, lse, static_cast<const T *>(dout), static_cast<T *>(dq), stat,
                       rpb_partial, p.H, p.W, p.heads, p.B, tiles_y, us.units, us.splits, us.gd, p.D == kHalfDim ? 1 : 0);
    return hipGetLastError();
}

// ---- part 2: key patches -> dk, dv -------------------------------------------------------------
//
// A workgroup owns a 16 x 8 key tile (eight waves, one 4 x 4 key patch each), keeps its position and head
// and walks a range of the batch.  The queries that see any key of the tile form a rectangle of at most
// (8 + K-1) x (16 + K-1) positions; per plane their q and dout vectors reach LDS by direct loads in the
// natural layout, their log-sum-exp and delta as pairs.  A patch takes its part of the rectangle in 4 x 4 blocks of
// queries, four rows at a time from the first row that sees it (rows past the last are masked):
//   S = Q_blk K^T, dP = dout_blk V^T         (queries as 16-byte A operands, the lane's key as B operand)
//   P = exp2(log2e (S' - lse)), dS = P (dP - delta)   per result; a lane holds 4 neighbouring queries of a row for its key
//   dv^T += dout_blk^T P, dk^T += Q_blk^T dS the half-depth MFMA (q / dout through the transposing LDS read)
// The bias of (query, key) depends on their offset only; per block a lane needs four neighbouring cells
// of one table row.  The table is kept in LDS mirrored left to right and in four copies shifted by one
// element each, so that every such run of four starts on an 8-byte boundary in one of them, and with a row of -inf below it
// that stands in for the rows of queries that do not see the lane's key; columns are masked by a packed addition.
// Why 4 x 4 blocks: 9 of them hold what an interior patch meets at K = 7 (4 at K = 3 and 5, 9 at K = 9), where rows of 16 columns took 10 (6, 8
// and 12), and the blocks of four rows share a lane's bias row, masks and addresses (immediate offsets between them).  lse and delta of a row's
// 16 columns are one LDS read, handed to the results by a row broadcast in the instruction that subtracts them.  The images' rows end 32 bytes
// behind their last position and the transposing reads take 32 contiguous bytes of a position: bank conflicts 4.4e6 -> 0.6e6, LDS busy 13e6 -> 5e6
// cycles, vector instructions 18.1e6 -> 12.0e6 a launch (64 x 2 x 56 x 56, K = 7, fp16).
// us, before / now, 56 x 56 x 2 x 64 unless said: fp16 K = 3 34.8 / 32.0, K = 5 42.0 / 32.8, K = 7 49.5 / 41.9, K = 9 78.5 / 66.5; bf16 K = 7 64.2 / 51.2;
// 14 x 14 x 8 x 128, K = 7, fp16 31.8 / 27.1, bf16 39.8 / 31.2.  The loads and stores alone take 27 us at the first shape (5.6 TB/s of
// compulsory traffic): what is above that is arithmetic that the other workgroups' loads do not cover.  Two buffers and a 16 x 16 tile per
// workgroup of 16 waves (one per compute unit) were no faster (48 us): four waves per SIMD do not fill the vector units.
// COMPACT: images sized for the rectangle of a tile away from the far border, (8 + K-1) x (16 + K-1) positions
// (three workgroups per compute unit); next to the far border the clamped queries reach R positions
// further, and a map with such tiles takes the larger images (two workgroups per compute unit).
template <typename T, int K, bool COMPACT>
struct FbwdKvCfg {
    static constexpr int R = K / 2;
    static constexpr int PWI = K + R + 3;   // query rows / columns that can see a 4 x 4 key patch
    static_assert(PWI <= 16, "four blocks of columns hold K + R + 3 <= 16");
    static constexpr int STRIPS = 2;
    static constexpr int WAVES = 4 * STRIPS;
    static constexpr int TY = 4 * STRIPS;
    // CHUNKED (K = 9): the images hold 16 rows of the rectangle at a time.  A rectangle of up to 20 rows (tiles next to
    // the far border) is taken in two chunks, its first 16 rows and its last 16 (the rows they share are used from the
    // first), so that two workgroups still share a compute unit; the accumulators stay in registers across them.
    static constexpr bool CHUNKED = K > 7;
    static_assert(!CHUNKED || !COMPACT, "the chunked images are always the wide ones");
    static constexpr int kRowsMax = TY + K - 1 + (COMPACT ? 0 : R);   // rows of a rectangle, at most
    static constexpr int RH = CHUNKED ? 16 : kRowsMax, RW = (kTileX + K - 1 + (COMPACT ? 0 : R) + 1) & ~1;   // the images (rows of an even number of positions)
    static_assert(kRowsMax <= 2 * RH, "two chunks");
    static constexpr int NB = 2 * K - 1;
    static constexpr int kThreads = kWave * WAVES;
    // (a row ends 32 bytes behind its last position: the operand reads of four rows and the transposing reads of two then meet every bank once)
    using XHalo = HaloDma<T, RH, RW, WAVES, 2>;
    static_assert(RW % 2 == 0, "rows start 8 or 40 banks from each other");
    // A patch takes its rows four at a time: the last four may reach kOver rows past the images' last (COMPACT: see kv_rows_fit), and the
    // columns of a patch, which starts in column 12 at most, 28 - RW positions past the last of them
    static constexpr int kOver = COMPACT ? 2 : 3;
    static constexpr int kXBytes = (RH + kOver) * XHalo::kRowBytes + (28 - RW) * Traits<T>::kKeyBytes;
    static_assert(RW <= 28, "columns");
    static constexpr int kSWords = RH * RW * 2;                             // (lse, delta) per position
    static constexpr int kSItems = (kSWords + kWave - 1) / kWave;           // 64-lane loads
    static constexpr int kSPerWave = (kSItems + WAVES - 1) / WAVES;
    static constexpr int kSBytes = ((RH + kOver) * RW + 28 - RW) * 8;
    static_assert(kXBytes % 16 == 0 && kSBytes % 16 == 0, "cleared in 16-byte pieces");
    static constexpr int BP = K > 7 ? 28 : 24;                      // row pitch (elements) of a bias copy (a multiple of 4)
    static_assert(NB + 3 + 3 + 3 < BP, "a shifted run of four stays inside its row");
    static constexpr int kBiasCopy = (NB + 1) * BP * 2;             // (the last row: -inf)
    static constexpr int kBiasBytes = 4 * kBiasCopy + 32;           // runs of masked columns go on behind a row
    static constexpr int kLdsBytes = 2 * kXBytes + kSBytes + kBiasBytes;
    static constexpr int kLdsAlloc = (kLdsBytes + 511) / 512 * 512;
    static constexpr int kWgPerCu = (160 * 1024) / kLdsAlloc < 3 ? (160 * 1024) / kLdsAlloc : 3;
    static_assert(kWgPerCu >= 2, "LDS");
    static constexpr int kWavesPerSimd = kWgPerCu * WAVES / 4;
};

typedef float f32v2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32v2 __attribute__((ext_vector_type(2)));
// two fp16 additions (written out: from a vector addition the compiler makes two, and two registers of what is kept)
__device__ __forceinline__ f16x2 add_packed(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_pk_add_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return __builtin_bit_cast(f16x2, r);
}
// x of lane C of the lane's group of 16, in all of them (a modifier of the instruction that uses it)
template <int C> __device__ __forceinline__ float column(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x150 + C, 0xf, 0xf, true));
}

template <typename T, int K, bool COMPACT>
__global__ __launch_bounds__(512, (FbwdKvCfg<T, K, COMPACT>::kWavesPerSimd)) void fbwd_kv_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ rpb, float scale,
    const float *__restrict__ stat, const T *__restrict__ dout, T *__restrict__ dk,
    T *__restrict__ dv, int H, int W, int heads, int nb, int tiles_y, int units, int splits, GridDecode gd, int half_dim, RpbPartials bias_grad, int own_blocks) {
    // Workgroups from own_blocks on add up the query-patch kernel's partial bias gradients (there are none without a bias gradient).
    // stat: the log-sum-exp of every query and its delta, as the query-patch kernel left them
    using C = FbwdKvCfg<T, K, COMPACT>;
    using XHalo = typename C::XHalo;
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr int KB = Traits<T>::kKeyBytes;
    extern __shared__ __align__(16) char lds[];
    if ((int)blockIdx.x >= own_blocks) {
        static_assert(C::kLdsBytes >= kRpbFinalLdsBytes, "LDS");
        rpb_final_block<C::kThreads>(bias_grad, blockIdx.x - own_blocks, lds_addr(lds));
        return;
    }

    const int wg = xcd_contiguous_block(blockIdx.x, own_blocks);
    if (wg >= units * splits) return;
    const WorkItem work = decode_work(wg, heads, tiles_y, splits, gd);
    const int head = work.head;
    const int b_begin = work.b_begin, b_end = work.b_end;
    if (b_begin >= b_end) return;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane & 15, g = lane >> 4, ky = n >> 2, kx = n & 3;
    const int lds0 = lds_addr(lds);
    const int q0 = lds0, l0 = lds0 + 2 * C::kXBytes, bias0 = l0 + C::kSBytes;   // q and dout of the rectangle; (lse, delta); bias copies

    // everything the loads do not write must hold finite numbers (it only ever meets P = 0)
    for (int i = tid * 16; i < C::kLdsBytes - C::kBiasBytes; i += C::kThreads * 16) *lds_ptr<u32x4>(lds0 + i) = u32x4{0u, 0u, 0u, 0u};
    // bias copies: copy s holds B[u][v] (see bias_to_f16) at element u * BP + (NB-1 - v) + 3 + s, zeros elsewhere, -inf in row NB
    for (int i = tid; i < C::kBiasBytes / 2; i += C::kThreads) {
        const int s = i / ((C::NB + 1) * C::BP), rest = i - s * ((C::NB + 1) * C::BP);
        const int u = rest / C::BP, col = rest - u * C::BP;
        const int vv = C::NB - 1 - (col - 3 - s);
        f16_t val = u == C::NB ? (f16_t)-INFINITY : (f16_t)0.f;
        if (rpb != nullptr && s < 4 && u < C::NB && (unsigned)vv < (unsigned)C::NB) val = bias_to_f16(rpb[((size_t)head * C::NB + u) * C::NB + vv]);
        *lds_ptr<f16_t>(bias0 + i * 2) = val;
    }

    const int ty0 = work.ty * C::TY, tx0 = work.tx * kTileX;
    const int ty1 = ty0 + C::TY - 1 < H - 1 ? ty0 + C::TY - 1 : H - 1;
    const int ry0 = inv_first(ty0, H, K), rx0 = inv_first(tx0, W, K);   // the rectangle (fits kRowsMax x RW: checked by the host)
    const int nrows = inv_last(ty1, H, K) - ry0 + 1;
    const int nch = C::CHUNKED && nrows > C::RH ? 2 : 1;   // chunks of the rectangle
    const int org1 = nrows - C::RH;                        // first rectangle row of the second chunk

    // loads of one plane
    XHalo xhalo;
    xhalo.init(wave, lane);
    int xoff[XHalo::PER_WAVE];
    // (half_dim: 16-channel heads; see kHalfDimChunks)
    const int pitch = half_dim ? KB / 2 : KB, chunk_mask = half_dim ? kHalfDimChunks : 3;
    xhalo.offsets(H, W, ry0, rx0, xoff, pitch, chunk_mask);
    int soff[C::kSPerWave];   // this lane's words of the pairs, clamped into the map (-1: nothing)
#pragma unroll
    for (int i = 0; i < C::kSPerWave; ++i) {
        const int w = (wave + i * C::WAVES) * kWave + lane, pos = w >> 1;
        const int rr = pos / C::RW, cc = pos - rr * C::RW;
        int y = ry0 + rr, x = rx0 + cc;
        y = y < H - 1 ? y : H - 1;
        x = x < W - 1 ? x : W - 1;
        soff[i] = w < C::kSWords ? (y * W + x) * 8 + (w & 1) * 4 : -1;
    }

    const int strip = wave >> 2, p = patch_of_wave(wave);
    const int sy0 = ty0 + 4 * strip, px0 = tx0 + 4 * p;   // this wave's key patch
    const bool active = sy0 < H && px0 < W;
    const int jy = sy0 + ky, jx = px0 + kx;                // this lane's key
    const bool key_ok = jy < H && jx < W;
    const int cy = jy < H ? jy : H - 1, cx = jx < W ? jx : W - 1;
    const int oqy = inv_first(sy0 < H ? sy0 : H - 1, H, K), oqx = inv_first(px0 < W ? px0 : W - 1, W, K);
    const int sy3 = sy0 + 3 < H - 1 ? sy0 + 3 : H - 1, px3 = px0 + 3 < W - 1 ? px0 + 3 : W - 1;
    const int nrow = active ? inv_last(sy3, H, K) - oqy + 1 : 0;         // rows and blocks of columns that see the patch
    const int ncol = active ? (inv_last(px3, W, K) - oqx + 4) >> 2 : 0;
    const int row0 = oqy - ry0, col0 = oqx - rx0;
    // lane-constant address parts inside four rows of the rectangle
    const int arow = q0 + (n >> 2) * XHalo::kRowBytes + (col0 + (n & 3)) * KB + g * 16;   // A operand: query n of a block, bytes [16g, 16g+16)
    const int atr = q0 + g * XHalo::kRowBytes + (col0 + (n >> 2)) * KB + (n & 3) * 8;     // transposing read: half hf holds channels 16 hf .. 16 hf + 15
    const int srow = l0 + (g * C::RW + col0 + n) * 8;                                     // pair of column n of row g
    // which queries see the lane's key: y_count rows (none for a lane without a key), counted so that a block's first row is the lane's row g - y_first ...
    const int key_first = inv_first(cy, H, K), y_first = key_first - oqy - g, y_count = key_ok ? inv_last(cy, H, K) - key_first + 1 : 0;
    // ... and columns, as what is added to the bias of two of them
    const int x_first = inv_first(cx, W, K) - oqx, x_count = inv_last(cx, W, K) - oqx + 1 - x_first;
    auto mask_of = [&](int c) {
        return ((unsigned)(c - x_first) < (unsigned)x_count ? 0u : 0xfc00u) | ((unsigned)(c + 1 - x_first) < (unsigned)x_count ? 0u : 0xfc000000u);
    };
    uint32_t colmask[4][2];
#pragma unroll
    for (int c = 0; c < 16; c += 2) colmask[c >> 2][(c >> 1) & 1] = mask_of(c);
    // bias: row u = jy - iy + K-1 of the table, mirrored columns NB-1 - (jx - ix + K-1) = vm0 + c
    int vm0 = K - 1 - (cx - oqx);
    vm0 = vm0 < -3 ? -3 : vm0;   // (outside the table only where nothing meets)
    const int shift = (-(vm0 + 3)) & 3;
    // of the first row that sees the key; the rows that follow lie in front of it (8-byte aligned)
    const int cbase = bias0 + shift * C::kBiasCopy + (vm0 + 3 + shift) * 2 + (cy - key_first + K - 1) * (C::BP * 2);
    const int no_row = bias0 + C::NB * (C::BP * 2);

    const size_t plane_px = (size_t)H * W;
    const unsigned key_off = (unsigned)((cy * W + cx) * pitch);   // (a plane is smaller than 2^31 bytes)
    workgroup_sync();

    for (int b = b_begin; b < b_end; ++b) {
        const size_t plane = (size_t)b * heads + head;
        // the lane's key and value: bytes [16g, 16g+16) (B operands)
        const size_t plane_off = plane * plane_px * pitch;
        const unsigned koff = key_off + (g & chunk_mask) * 16;
        const bool upper = half_dim && g >= 2;   // lanes whose channels a 16-channel head does not have
        const u32x4 kload = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(k) + plane_off + koff);
        const u32x4 vload = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(v) + plane_off + koff);
        const u32x4 kreg = upper ? u32x4{0u, 0u, 0u, 0u} : kload, vreg = upper ? u32x4{0u, 0u, 0u, 0u} : vload;
        f32x4 ak[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};   // dk^T, dv^T: channels 8g + 4 hf + r of the lane's key
        f32x4 av[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
        for (int c = 0; c < nch; ++c) {
        if (b > b_begin || c > 0) workgroup_sync();   // the previous images are no longer read
        // rows of the rectangle in the images: [org, org + RH); the second chunk lies inside the map as a whole
        const int org = c ? org1 : 0;
        {
            int xo[XHalo::PER_WAVE];
#pragma unroll
            for (int i = 0; i < XHalo::PER_WAVE; ++i) xo[i] = xoff[i] >= 0 ? xoff[i] + org * W * pitch : -1;
            XHalo::issue_at(reinterpret_cast<const char *>(q) + plane * plane_px * pitch, xo, q0, wave);
            XHalo::issue_at(reinterpret_cast<const char *>(dout) + plane * plane_px * pitch, xo, q0 + C::kXBytes, wave);
        }
#pragma unroll
        for (int i = 0; i < C::kSPerWave; ++i)
            if (soff[i] >= 0)
                global_to_lds_4(reinterpret_cast<const char *>(stat) + plane * plane_px * 8, (unsigned)(soff[i] + org * W * 8), l0 + (wave + i * C::WAVES) * kWave * 4);
        wait_global_loads();
        workgroup_sync();
        if (!active) continue;

        // the block of columns 4 CB .. 4 CB + 3 of four rows (offset of their first in the images; the lane's row of the bias table; the pair of column n)
        auto block = [&](auto cb, int pos, int brow, const f32v2 &st) {
            constexpr int CB = decltype(cb)::value;
            const int ra = arow + pos + CB * 4 * KB, rt = atr + pos + CB * 4 * KB;
            const u32x4 aq = *lds_ptr<u32x4>(ra), ad = *lds_ptr<u32x4>(ra + C::kXBytes);
            const u32v2 b4 = *lds_ptr<u32v2>(brow + CB * 8);
            const f32x4 sacc = mfma_16x16x32<T>(aq, kreg, f32x4{0.f, 0.f, 0.f, 0.f});
            const f32x4 pacc = mfma_16x16x32<T>(ad, vreg, f32x4{0.f, 0.f, 0.f, 0.f});
            float pw[4], ds[4];
            auto two = [&](auto half) {
                constexpr int h = decltype(half)::value, c = 4 * CB + 2 * h;   // columns c, c + 1
                const f16x2 bias = add_packed(h ? b4.y : b4.x, colmask[CB][h]);   // -inf outside the window
                pw[2 * h] = __builtin_amdgcn_exp2f((__builtin_fmaf(scale, sacc[2 * h], (float)bias[0]) - column<c>(st.x)) * kLog2e);
                pw[2 * h + 1] = __builtin_amdgcn_exp2f((__builtin_fmaf(scale, sacc[2 * h + 1], (float)bias[1]) - column<c + 1>(st.x)) * kLog2e);
                ds[2 * h] = pw[2 * h] * (pacc[2 * h] - column<c>(st.y));
                ds[2 * h + 1] = pw[2 * h + 1] * (pacc[2 * h + 1] - column<c + 1>(st.y));
            };
            two(IntC<0>{});
            two(IntC<1>{});
            if constexpr (Traits<T>::kDtype == NA2D_BF16) __builtin_amdgcn_sched_barrier(0);   // (one sum after the other: the registers)
            auto sum = [&](f32x4 (&acc)[2], const float (&w)[4], int at) {
                const u32x2 t[2] = {lds_read_tr16(at), lds_read_tr16(at + 32)};
                const uint32_t w0 = pack2_t<T>(w[0], w[1]), w1 = pack2_t<T>(w[2], w[3]);
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) acc[hf] = mfma_16x16x16<T>(t[hf].x, t[hf].y, w0, w1, acc[hf]);
                if constexpr (Traits<T>::kDtype == NA2D_BF16) {
                    // bf16 keeps 8 significant bits: second operands carry the rounding remainders of P and dS
                    const uint32_t l0 = pack_remainders(w0, w[0], w[1]), l1 = pack_remainders(w1, w[2], w[3]);
#pragma unroll
                    for (int hf = 0; hf < 2; ++hf) acc[hf] = mfma_16x16x16<T>(t[hf].x, t[hf].y, l0, l1, acc[hf]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            sum(av, pw, rt + C::kXBytes);
            sum(ak, ds, rt);
        };
        // this chunk's part of the rows that see the patch: rectangle rows below RH in the first chunk, the others in
        // the second
        const int lo = c ? (C::RH - row0 > 0 ? C::RH - row0 : 0) : 0;
        const int hi = (nch == 2 && c == 0) ? (nrow < C::RH - row0 ? nrow : C::RH - row0) : nrow;
        int count = y_count;
        if constexpr (C::CHUNKED) {   // (rows of the second chunk stay away from the first: there are none of them in its images)
            const int left = hi - (y_first + g);
            count = key_ok && left < count ? left : count;
        }
        auto rows = [&](auto cols) {   // (a loop for each number of block columns: the accumulators stay where they are)
            constexpr int COLS = decltype(cols)::value;
            if (C::CHUNKED && lo >= hi) return;   // (a patch that is in the map is seen by at least one row)
            int row = lo;
            do {
                const int in = row - y_first;   // the lane's row of the block, counted from the first that sees the key
                const int brow = (unsigned)in < (unsigned)count ? __mul24(in, -(C::BP * 2)) + cbase : no_row;
                int at = row0 + row - org;
                asm volatile("" : "+s"(at));   // (no second set of addresses that runs along)
                const f32v2 st = *lds_ptr<f32v2>(srow + at * (C::RW * 8));
                block(IntC<0>{}, at * XHalo::kRowBytes, brow, st);
                block(IntC<1>{}, at * XHalo::kRowBytes, brow, st);
                if constexpr (COLS > 2) block(IntC<2>{}, at * XHalo::kRowBytes, brow, st);
                if constexpr (COLS > 3) block(IntC<3>{}, at * XHalo::kRowBytes, brow, st);
                row += 4;
            } while (row < hi);
        };
        if (ncol <= 2) rows(IntC<2>{});   // (one: the second is masked)
        else if (ncol == 3) rows(IntC<3>{});
        else rows(IntC<4>{});
        }   // chunks
        settle_products<2>(ak);
        settle_products<2>(av);
        if (key_ok) {
            const unsigned o = key_off + g * 8;
            // channels 4g .. 4g + 3 of either half
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if (half_dim && hf) continue;
                *reinterpret_cast<u32v2 *>(reinterpret_cast<char *>(dk) + plane_off + o + hf * 32) = u32v2{pack2_t<T>(ak[hf][0] * scale, ak[hf][1] * scale), pack2_t<T>(ak[hf][2] * scale, ak[hf][3] * scale)};
                *reinterpret_cast<u32v2 *>(reinterpret_cast<char *>(dv) + plane_off + o + hf * 32) = u32v2{pack2_t<T>(av[hf][0], av[hf][1]), pack2_t<T>(av[hf][2], av[hf][3])};
            }
        }
    }
}

// Does the query rectangle of every 16 x 8 key tile fit rows x cols positions?
static bool kv_rect_fits(const Problem &p, int rows, int cols) {
    const int K = p.K, TY = 8;
    for (int ty0 = 0; ty0 < p.H; ty0 += TY) {
        const int ty1 = ty0 + TY - 1 < p.H - 1 ? ty0 + TY - 1 : p.H - 1;
        if (inv_last(ty1, p.H, K) - inv_first(ty0, p.H, K) + 1 > rows) return false;
    }
    for (int tx0 = 0; tx0 < p.W; tx0 += kTileX) {
        const int tx1 = tx0 + kTileX - 1 < p.W - 1 ? tx0 + kTileX - 1 : p.W - 1;
        if (inv_last(tx1, p.W, K) - inv_first(tx0, p.W, K) + 1 > cols) return false;
    }
    return true;
}

// Do the rows of every patch, taken in fours, end within two rows of the `rows` that its tile's rectangle has at most?
static bool kv_rows_fit(const Problem &p, int rows) {
    for (int sy = 0; sy < p.H; sy += 4) {
        const int first = inv_first(sy, p.H, p.K), last = inv_last(sy + 3 < p.H - 1 ? sy + 3 : p.H - 1, p.H, p.K);
        if (first - inv_first(sy & ~7, p.H, p.K) + ((last - first + 4) & ~3) > rows + 2) return false;
    }
    return true;
}

template <typename T, int K, bool COMPACT>
static hipError_t launch_fbwd_kv_c(const Problem &p, const void *q, const void *k, const void *v, const void *rpb,
                                   float scale, const float *stat, const void *dout, void *dk, void *dv,
                                   const RpbPartials &bias_grad, hipStream_t s) {
    using C = FbwdKvCfg<T, K, COMPACT>;
    const int tiles_x = (p.W + kTileX - 1) / kTileX, tiles_y = (p.H + C::TY - 1) / C::TY;
    const int units = tiles_x * tiles_y * p.heads;
    int splits = (256 * C::kWgPerCu) / units;
    splits = splits < 1 ? 1 : (splits < p.B ? splits : p.B);
    auto kern = fbwd_kv_kernel<T, K, COMPACT>;
    static LdsAllowed allowed;
    if (hipError_t e = allow_lds(kern, C::kLdsBytes, allowed); e != hipSuccess) return e;
    const int own_blocks = xcd_padded_grid(units * splits), last_sum = bias_grad.d_rpb ? p.heads * rpb_final_blocks(C::NB * C::NB) : 0;
    const bool along = launch_holds((long long)own_blocks + last_sum, C::kThreads);
    hipLaunchKernelGGL(kern, dim3(own_blocks + (along ? last_sum : 0)), dim3(C::kThreads), C::kLdsBytes, s,
                       static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
                       static_cast<const T *>(rpb), scale, stat, static_cast<const T *>(dout), static_cast<T *>(dk),
                       static_cast<T *>(dv), p.H, p.W, p.heads, p.B, tiles_y, units, splits, make_grid_decode(tiles_x, tiles_y, p.heads, p.B, splits),
                       p.D == kHalfDim ? 1 : 0, bias_grad, own_blocks);
    if (hipError_t e = hipGetLastError(); e != hipSuccess || along) return e;
    return launch_rpb_final_av(p, bias_grad.partial, bias_grad.d_rpb, fused_bwd_split(p), s);
}

template <typename T, int K>
static hipError_t launch_fbwd_kv_t(const Problem &p, const void *q, const void *k, const void *v, const void *rpb,
                                   float scale, const float *stat, const void *dout, void *dk, void *dv,
                                   const RpbPartials &bias_grad, hipStream_t s) {
    if constexpr (K > 7) {   // (chunked images: one size)
        return launch_fbwd_kv_c<T, K, false>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);
    } else {
        return kv_rect_fits(p, 8 + K - 1, kTileX + K - 1) && kv_rows_fit(p, 8 + K - 1)
                   ? launch_fbwd_kv_c<T, K, true>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s)
                   : launch_fbwd_kv_c<T, K, false>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);
    }
}

hipError_t launch_fbwd_kv(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale,
                          const float *stat, const void *dout, void *dk, void *dv, const float *rpb_partial, BiasOut d_rpb, hipStream_t s) {
    const AvRpbSplit sp = fused_bwd_split(p);
    const RpbPartials bias_grad{rpb_partial, d_rpb, sp.npos * sp.splits, (2 * p.K - 1) * (2 * p.K - 1)};
#define NA2D_FBKV_K(TT)                                                                                   \
    switch (p.K) {                                                                                        \
        case 3: return launch_fbwd_kv_t<TT, 3>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);      \
        case 5: return launch_fbwd_kv_t<TT, 5>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);      \
        case 7: return launch_fbwd_kv_t<TT, 7>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);      \
        case 9: return launch_fbwd_kv_t<TT, 9>(p, q, k, v, rpb, scale, stat, dout, dk, dv, bias_grad, s);      \
        default: return hipErrorInvalidValue;                                                             \
    }
    if (p.dtype == NA2D_F16) { NA2D_FBKV_K(f16_t) }
    if (p.dtype == NA2D_BF16) { NA2D_FBKV_K(bf16_t) }
#undef NA2D_FBKV_K
    return hipErrorInvalidValue;
}

// Is every 4-column key patch seen from at most 16 query columns (one MFMA block per rectangle row)?  Always so
// away from short axes (K + (K-1)/2 + 3 <= 16 columns); on an axis of at most 2K + 2 positions a patch can be seen
// from both clamped ends at once, and then it depends on the length.
static bool kv_patch_cols_fit(const Problem &p) {
    for (int px = 0; px < p.W; px += 4)
        if (inv_last(px + 3 < p.W - 1 ? px + 3 : p.W - 1, p.W, p.K) - inv_first(px, p.W, p.K) + 1 > 16) return false;
    return true;
}

// The second kernel sizes its images for key tiles that are next to at most one border per axis: a 16 x 8 tile
// whose query rectangle exceeds (8 + K-1 + R) x (16 + K-1 + R) positions (short axes, where a ragged tile is
// close to both borders) does not fit, and such maps take the unfused steps instead.
bool fused_bwd_supported(const Problem &p) {
    const int R = p.K / 2;
    return (p.D == kHeadDim || p.D == kHalfDim) && p.dtype != NA2D_F32 && p.K <= 9 && kv_patch_cols_fit(p) &&
           kv_rect_fits(p, 8 + p.K - 1 + R, kTileX + p.K - 1 + R);
}

AvRpbSplit fused_bwd_split(const Problem &p) {
    const int tiles_x = (p.W + kTileX - 1) / kTileX, tiles_y = (p.H + 7) / 8;
    const UnitSplit us = unit_split(tiles_x, tiles_y, p.heads, p.B);
    return AvRpbSplit{us.units / p.heads, us.splits};
}

hipError_t launch_fbwd_q(const Problem &p, const void *q, const void *k, const void *v, const void *rpb, float scale,
                         const float *lse, const void *dout, void *dq, float *stat, float *rpb_partial,
                         hipStream_t s) {
#define NA2D_FBQ_K(TT)                                                                                             \
    switch (p.K) {                                                                                                 \
        case 3: return launch_fbwd_q_t<TT, 3>(p, q, k, v, rpb, scale, lse, dout, dq, stat, rpb_partial, s);       \
        case 5: return launch_fbwd_q_t<TT, 5>(p, q, k, v, rpb, scale, lse, dout, dq, stat, rpb_partial, s);       \
        case 7: return launch_fbwd_q_t<TT, 7>(p, q, k, v, rpb, scale, lse, dout, dq, stat, rpb_partial, s);       \
        case 9: return launch_fbwd_q_t<TT, 9>(p, q, k, v, rpb, scale, lse, dout, dq, stat, rpb_partial, s);       \
        default: return hipErrorInvalidValue;                                                                      \
    }
    if (p.dtype == NA2D_F16) { NA2D_FBQ_K(f16_t) }
    if (p.dtype == NA2D_BF16) { NA2D_FBQ_K(bf16_t) }
#undef NA2D_FBQ_K
    return hipErrorInvalidValue;
}

}  // namespace na2d
