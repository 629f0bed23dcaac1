// The last sum of the bias gradient: d_rpb[h, cell] = sum over i < n of partial[h * n + i][cell], rows of rpb_cell_stride(cells) floats.
// A kernel of its own where the partials come from the last kernel of a call; where they are there before the last kernel starts, workgroups
// at the end of that kernel's grid do it (one launch less: about 4 us of GPU time and as much of the host's).
#pragma once

#include "na2d_kernels.hpp"
#include "na2d_mfma.hpp"

namespace na2d {

struct RpbPartials {
    const float *partial;
    BiasOut d_rpb;
    int n, cells;   // partials per head; cells of a head's table
};
struct __attribute__((packed, aligned(4))) RpbQuad {
    f32x4 v;
};
// A workgroup per head and 16 cells: four lanes own four neighbouring cells each (one 16-byte load per
// partial); 256 groups of four lanes take the partials in turn, eight loads in flight, and their sub-sums are added in group
// order (whatever the number of threads that stand for the groups).  The time is the latency of a group's loads, one behind the other from eight
// on, so few cells to a workgroup: with 64 of them 1 head of 1792 partials of 169 cells took 8.6 us, now 5.4; 2 heads of 1792 partials of 625 5.6, now 4.7.
constexpr int kRpbFinalLanes = 4, kRpbFinalGroups = 256, kRpbFinalLdsBytes = kRpbFinalGroups * kRpbFinalLanes * 16;
__host__ __device__ constexpr int rpb_final_blocks(int cells) { return (rpb_cell_stride(cells) / 4 + kRpbFinalLanes - 1) / kRpbFinalLanes; }   // per head

// block `block` of heads * rpb_final_blocks(cells); sub0: kRpbFinalLdsBytes of LDS
template <int THREADS> __device__ __forceinline__ void rpb_final_block(const RpbPartials &p, int block, int sub0) {
    static_assert(THREADS >= kWave && kRpbFinalGroups * kRpbFinalLanes % THREADS == 0, "groups");
    const int stride = rpb_cell_stride(p.cells), quad_blocks = rpb_final_blocks(p.cells), h = block / quad_blocks;
    const int lane = threadIdx.x % kRpbFinalLanes, cell0 = ((block - h * quad_blocks) * kRpbFinalLanes + lane) * 4;   // this lane's first cell
    for (int group = threadIdx.x / kRpbFinalLanes; group < kRpbFinalGroups; group += THREADS / kRpbFinalLanes) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        if (cell0 < stride) {
            const float *base = p.partial + (size_t)h * p.n * stride + cell0;
            constexpr int U = 8;   // loads in flight per lane; past the end they are skipped (adding 0 changes nothing)
            for (int i = group; i < p.n; i += U * kRpbFinalGroups) {
                f32x4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int iu = i + u * kRpbFinalGroups;
                    v[u] = iu < p.n ? reinterpret_cast<const RpbQuad *>(base + (size_t)iu * stride)->v : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int u = 0; u < U; ++u) acc += v[u];
            }
        }
        *lds_ptr<f32x4>(sub0 + (group * kRpbFinalLanes + lane) * 16) = acc;
    }
    workgroup_sync();
    // sixteen lanes of the first wave per cell quad: sixteen sub-sums each, then the sixteen
    if (threadIdx.x < kWave) {
        static_assert(kRpbFinalGroups == 16 * (kWave / kRpbFinalLanes), "sub-sums");
        const int part = threadIdx.x / kRpbFinalLanes;
        const auto sub = [&](int w) { return *lds_ptr<f32x4>(sub0 + ((part * 16 + w) * kRpbFinalLanes + lane) * 16); };
        f32x4 t = sub(0);
        for (int w = 1; w < 16; ++w) t += sub(w);
#pragma unroll
        for (int m = kRpbFinalLanes; m < kWave; m *= 2)
#pragma unroll
            for (int c = 0; c < 4; ++c) t[c] += __shfl_xor(t[c], m);
        if (part == 0 && cell0 < p.cells) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (cell0 + c < p.cells) p.d_rpb.store((size_t)h * p.cells + cell0 + c, t[c]);
        }
    }
}

}  // namespace na2d
