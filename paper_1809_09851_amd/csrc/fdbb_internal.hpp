// Host-side glue between the C ABI (fdbb_api.hip) and the kernel
// translation units.  Each kernel unit returns the address of the template
// instance for (dim, dtype, points per thread).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "euler_tiles.hpp"

namespace fdbb {

// Device image of one batch task: the operation's arguments plus what the
// batch kernels need to pick the tile function and its parts.
struct TaskDev {
    Args a;
    int32_t op;
    int32_t dim;
    int32_t dtype;
    int32_t groups;      // sets of parts a tile is dealt in (1: the whole tile)
    int64_t first_unit;  // the task's entry of the prefix sums
};

// Points of one span of a split launch (see Split).
constexpr int64_t kSpanPoints = 131072;

// The parts of set k of a fused pass or flux Jacobian dealt in `groups` sets:
// the whole tile, one direction each, or all rows and then one direction's
// blocks each.
template <int D>
__device__ __forceinline__ uint32_t batch_mask(int groups, uint32_t k)
{
    constexpr uint32_t dirs = all_directions<D>;
    if (groups == 1) return dirs << kPartFields | dirs;
    if (groups == D) return (1u << kPartFields | 1u) << k;
    return k == 0 ? dirs << kPartFields : 1u << (k - 1);
}

// Largest workgroup of the kernels that stage Jacobian blocks (the fused
// kernel and the batch kernel).  Bounding them at 256 threads lets the
// compiler give each thread up to 256 registers, so the staged blocks never
// spill; their occupancy is set by LDS anyway.
constexpr int kMaxBlockStaged = 256;

// Kernel families (a family covers one or more public ops).
enum Family : int {
    kFamCons2Prim = 0,
    kFamPrim2Cons,
    kFamEos,
    kFamFlux,
    kFamRiemann,
    kFamCons2Char,
    kFamChar2Cons,
    kFamFused,  // fused pass and flux Jacobian (F and R NULL)
    kFamAdjoint,
    kFamVmag2,
    kFamEigen,      // eigenvector blocks (staged like the Jacobian)
    kFamCharApply,  // products with L or R of one direction
    kFamRoe,        // Roe-averaged state of two states
    kFamEosPvt,     // p, c and T of the general EOS entry
    kFamViscous,    // viscous flux tensor
    kNumFamilies
};

// Single-operation kernels: void k(Args a, int64_t ntiles), and a third
// argument Split for the fused pass and the eigenvector blocks.  nt selects
// non-temporal output stores.
const void *kernel_pointwise(int family, int dim, int dtype, int ppt, bool nt);
const void *kernel_char(int family, int dim, int dtype, int ppt, bool nt);
const void *kernel_fused(int dim, int dtype, int ppt, bool nt, bool rows);  // rows: flux or invariants too
const void *kernel_adjoint(int dim, int dtype, int ppt, bool nt);
const void *kernel_eigen(int family, int dim, int dtype, int ppt, bool nt);

// Batch kernels: void k(const TaskDev*, const int64_t* prefix, const int64_t*
// header).  header = {ntasks, nunits}; prefix has ntasks + 1 entries,
// prefix[b] = first unit of task b.  ppt 1, 2, 4 or 8 (the fused kernel: 1, 2
// or 4, else null); store_mode 0 regular, 1 nt, 2 nt + sc1.  The general
// kernel takes whole tiles (one unit each) of any batchable op; the fused one
// lists of block-writing tasks of one dim and storage type.
const void *kernel_batch(int ppt, int store_mode);
const void *kernel_batch_fused(int dim, int dtype, int ppt, int store_mode);

// The allocation-free batch entry point's fixed task table: room for
// kNoAllocMaxTasks tasks in the layout of a plan's table (header, tile
// prefix sums, task images).
constexpr int kNoAllocMaxTasks = 1024;
constexpr size_t kNoAllocBytes =
    (((2 + (size_t)kNoAllocMaxTasks + 1) * sizeof(int64_t) + 63) & ~(size_t)63) + (size_t)kNoAllocMaxTasks * sizeof(TaskDev);

// Device address of that table on the current device (looked up with
// hipGetSymbolAddress on a device's first call, then cached); 0 or a
// hipError_t.
int batch_scratch(void **ptr);

}  // namespace fdbb
