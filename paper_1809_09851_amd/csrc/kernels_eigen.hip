// Characteristic decomposition kernels: eigenvector blocks of every
// direction (staged through LDS like the Jacobian) and products with L or R
// of one direction.
#include "fdbb_internal.hpp"

namespace fdbb {

// Bound by how DRAM takes the output streams, like the fused pass: in 3D one
// of the 2D block arrays per workgroup, in spans of tiles, with few waves
// resident.  Against all six arrays from one workgroup: FP64 1 000 003 points
// 225 -> 190 us (6.5 TB/s), 4 000 037 857 -> 765 us; FP32 4 000 037 points
// 437 -> 376 us.
template <int D, typename T, int P, int NT>
__global__ __launch_bounds__(kMaxBlockStaged) void k_eigen(Args a, int64_t ntiles, Split sp)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *lds = reinterpret_cast<T *>(smem);
    const int64_t tile_pts = (int64_t)blockDim.x * P;
    const uint32_t units = (uint32_t)ntiles * sp.groups;
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const Unit w = unit_of(sp.groups, sp.span, (uint32_t)ntiles, u);
        tile_eigen<D, T, P, NT>(a, w.tile * tile_pts, sp.mask[w.set], lds);
    }
}

template <int D, typename T, int P, int NT>
__global__ __launch_bounds__(1024) void k_char_apply(Args a, int64_t ntiles)
{
    const int64_t tile_pts = (int64_t)blockDim.x * P;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) tile_char_apply<D, T, P, NT>(a, t * tile_pts);
}

template <int FAM, int D, typename T, int NT>
static const void *pick_p(int ppt)
{
    if constexpr (FAM == kFamEigen) {
        switch (ppt) {
        case 1: return (const void *)&k_eigen<D, T, 1, NT>;
        case 2: return (const void *)&k_eigen<D, T, 2, NT>;
        case 4: return (const void *)&k_eigen<D, T, 4, NT>;
        default: return nullptr;
        }
    } else {
        switch (ppt) {
        case 1: return (const void *)&k_char_apply<D, T, 1, NT>;
        case 2: return (const void *)&k_char_apply<D, T, 2, NT>;
        case 4: return (const void *)&k_char_apply<D, T, 4, NT>;
        default: return nullptr;
        }
    }
}

template <int FAM, int D, typename T>
static const void *pick_p(int ppt, bool nt)
{
    // eigenvector blocks stream with nt + sc1, but in 3D FP64 (four resident
    // waves) and the products with nt
    constexpr int streaming = FAM == kFamEigen && !(D == 3 && sizeof(T) == 8) ? kStoreNTSc1 : kStoreNT;
    return nt ? pick_p<FAM, D, T, streaming>(ppt) : pick_p<FAM, D, T, kStoreRegular>(ppt);
}

template <int FAM>
static const void *pick(int dim, int dtype, int ppt, bool nt)
{
    if (dtype == 0) {
        if (dim == 1) return pick_p<FAM, 1, double>(ppt, nt);
        if (dim == 2) return pick_p<FAM, 2, double>(ppt, nt);
        if (dim == 3) return pick_p<FAM, 3, double>(ppt, nt);
    } else {
        if (dim == 1) return pick_p<FAM, 1, float>(ppt, nt);
        if (dim == 2) return pick_p<FAM, 2, float>(ppt, nt);
        if (dim == 3) return pick_p<FAM, 3, float>(ppt, nt);
    }
    return nullptr;
}

const void *kernel_eigen(int family, int dim, int dtype, int ppt, bool nt)
{
    if (family == kFamEigen) return pick<kFamEigen>(dim, dtype, ppt, nt);
    if (family == kFamCharApply) return pick<kFamCharApply>(dim, dtype, ppt, nt);
    return nullptr;
}

}  // namespace fdbb
