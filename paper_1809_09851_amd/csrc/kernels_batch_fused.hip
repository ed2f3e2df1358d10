// Batch kernel for lists whose tasks all write K x K blocks (fused passes and
// flux Jacobians) of one dim and storage type: the fused pass's kernel with a
// task lookup in front.
//
// Bound, like the fused pass, by how DRAM takes the output streams, so a
// workgroup takes one unit (one set of a tile's parts), few waves are
// resident and the hardware dispatcher deals the units; the general batch
// kernel's persistent workgroups, at the registers of its most demanding op,
// keep every stream of a tile open.  Fused pass over 96 uneven 3D FP64 blocks
// of 16.3 M points (13.3 GB): 2570 us (5.2 TB/s) with the general kernel, 2330
// (5.7) with this one.
#include "fdbb_internal.hpp"

namespace fdbb {

// Last task whose first unit is <= u, found by the whole wave: one load per
// 64-fold narrowing (one load up to 64 tasks, two up to 4096), where a
// bisection would chain a load per halving in front of every unit.
__device__ __forceinline__ int task_of(const int64_t *__restrict__ prefix, int ntasks, int64_t u)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, len = ntasks;
    while (len > 1) {
        const int step = (len + kWave - 1) / kWave;
        const int at = lane * step;
        const uint64_t le = __ballot(at < len && prefix[lo + at] <= u);
        const int k = 63 - __builtin_clzll(le | 1u);
        lo += k * step;
        len = len - k * step < step ? len - k * step : step;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

template <int D, typename T, int P, int NT>
__global__ __launch_bounds__(kMaxBlockStaged) void k_batch_fused(const TaskDev *__restrict__ tasks,
                                                                 const int64_t *__restrict__ prefix,
                                                                 const int64_t *__restrict__ header)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *lds = reinterpret_cast<T *>(smem);
    const int ntasks = (int)header[0];
    const int64_t units = header[1];
    const int64_t tile_pts = (int64_t)blockDim.x * P;
    const uint32_t span = (uint32_t)(kSpanPoints / tile_pts);  // tiles hold at most 1024 points
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const TaskDev &td = tasks[task_of(prefix, ntasks, u)];
        const uint32_t ntiles = (uint32_t)((td.a.n + tile_pts - 1) / tile_pts);
        const Unit w = unit_of((uint32_t)td.groups, span, ntiles, (uint32_t)(u - td.first_unit));
        tile_fused<D, T, P, NT>(td.a, w.tile * tile_pts, batch_mask<D>(td.groups, w.set), lds);
    }
}

template <int D, typename T, int NT>
static const void *pick_p(int ppt)
{
    switch (ppt) {
    case 1: return (const void *)&k_batch_fused<D, T, 1, NT>;
    case 2: return (const void *)&k_batch_fused<D, T, 2, NT>;
    case 4: return (const void *)&k_batch_fused<D, T, 4, NT>;
    default: return nullptr;
    }
}

template <int D, typename T>
static const void *pick_nt(int ppt, int store_mode)
{
    switch (store_mode) {
    case 0: return pick_p<D, T, kStoreRegular>(ppt);
    case 1: return pick_p<D, T, kStoreNT>(ppt);
    case 2: return pick_p<D, T, kStoreNTSc1>(ppt);
    default: return nullptr;
    }
}

const void *kernel_batch_fused(int dim, int dtype, int ppt, int store_mode)
{
    if (dtype == 0) {
        if (dim == 1) return pick_nt<1, double>(ppt, store_mode);
        if (dim == 2) return pick_nt<2, double>(ppt, store_mode);
        if (dim == 3) return pick_nt<3, double>(ppt, store_mode);
    } else {
        if (dim == 1) return pick_nt<1, float>(ppt, store_mode);
        if (dim == 2) return pick_nt<2, float>(ppt, store_mode);
        if (dim == 3) return pick_nt<3, float>(ppt, store_mode);
    }
    return nullptr;
}

}  // namespace fdbb
