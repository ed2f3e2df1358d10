// Fused pass kernel: flux tensor, flux Jacobian blocks (staged through LDS)
// and Riemann invariants of the same state.  The flux-Jacobian entry point
// runs this kernel with the flux and invariant outputs NULL.
//
// Bound by how DRAM takes the output streams: 22 field rows and three block
// streams in 3D, 776 of the 816 bytes per point FP64.  Where the blocks do
// not fit in the last-level cache, a 3D workgroup therefore writes one set of
// its tile's parts (Split, chosen by split_of on the host): in FP64 one
// direction's rows and blocks, in FP32, where a row's run is half as long,
// one direction's blocks or all rows, and that up to 512 MiB of blocks (1.79 M
// points) only.  Spans of tiles go through one set after the other, few waves
// are resident (the launch reserves LDS), and the state that a later set
// reads again comes from the last-level cache.  FP32 beyond takes whole tiles
// with few waves resident.  Against one workgroup per tile at the best shape,
// on the same buffers: FP64 1 000 003 points 144 -> 125 us, 4 000 037 535 ->
// 513 us, 2^24 2410 -> 2340 us (5.85 TB/s); FP32 apart 1 000 003 points 69 ->
// 64 us, 1 500 001 105 -> 94 us, whole tiles 2 500 009 182 -> 178 us, 2^24
// over three sets of arrays 1213 -> 1173 us.
#include "fdbb_internal.hpp"

namespace fdbb {

template <int D, typename T, int P, int NT>
__global__ __launch_bounds__(kMaxBlockStaged) void k_fused(Args a, int64_t ntiles, Split sp)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *lds = reinterpret_cast<T *>(smem);
    const int64_t tile_pts = (int64_t)blockDim.x * P;
    const uint32_t units = (uint32_t)ntiles * sp.groups;
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const Unit w = unit_of(sp.groups, sp.span, (uint32_t)ntiles, u);
        tile_fused<D, T, P, NT>(a, w.tile * tile_pts, sp.mask[w.set], lds);
    }
}

template <int D, typename T, int NT>
static const void *pick_p(int ppt)
{
    switch (ppt) {
    case 1: return (const void *)&k_fused<D, T, 1, NT>;
    case 2: return (const void *)&k_fused<D, T, 2, NT>;
    case 4: return (const void *)&k_fused<D, T, 4, NT>;
    default: return nullptr;
    }
}

// Streaming flavour: nt for the 3D FP64 pass with rows (four resident waves:
// nt + sc1 ran 9 % slower), nt + sc1 for the rest (3D FP64 Jacobian 5 %, 2D
// FP64 pass 4 % faster than nt).
template <int D, typename T>
static const void *pick_p(int ppt, bool nt, bool rows)
{
    if (!nt) return pick_p<D, T, kStoreRegular>(ppt);
    if constexpr (D == 3 && sizeof(T) == 8)
        if (rows) return pick_p<D, T, kStoreNT>(ppt);
    return pick_p<D, T, kStoreNTSc1>(ppt);
}

const void *kernel_fused(int dim, int dtype, int ppt, bool nt, bool rows)
{
    if (dtype == 0) {
        if (dim == 1) return pick_p<1, double>(ppt, nt, rows);
        if (dim == 2) return pick_p<2, double>(ppt, nt, rows);
        if (dim == 3) return pick_p<3, double>(ppt, nt, rows);
    } else {
        if (dim == 1) return pick_p<1, float>(ppt, nt, rows);
        if (dim == 2) return pick_p<2, float>(ppt, nt, rows);
        if (dim == 3) return pick_p<3, float>(ppt, nt, rows);
    }
    return nullptr;
}

}  // namespace fdbb
