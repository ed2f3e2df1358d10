// C ABI of the library (declared in include/fdbb.h): host-side validation,
// launch configuration, kernel launches on the caller's stream, and the
// batch plans with their HIP graphs.
#include "../../include/fdbb.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "fdbb_internal.hpp"

using namespace fdbb;

namespace {

thread_local std::string g_last_error;

int fail(int status, const std::string &msg)
{
    g_last_error = msg;
    return status;
}

int fail_hip(hipError_t e, const char *what)
{
    return fail(FDBB_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

size_t elem_size(int dtype) { return dtype == FDBB_F64 ? 8 : 4; }

// ------------------------------------------------------------ device facts

struct DeviceInfo {
    int id = 0;
    int cus = 0;
    size_t lds_max = 0;
};

// Per-device facts, read once and then served without a lock: the first
// callers on a device may query concurrently, and all store the same values.
constexpr int kMaxDevices = 64;
std::atomic<int> g_dev_cus[kMaxDevices];
std::atomic<int64_t> g_dev_lds[kMaxDevices];

int device_info(DeviceInfo *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(FDBB_EHIP, "device index out of range");
    int cus = g_dev_cus[dev].load(std::memory_order_acquire);
    if (cus == 0) {
        int lds = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
        e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
        if (e != hipSuccess) return fail_hip(e, "hipDeviceGetAttribute");
        g_dev_lds[dev].store(lds, std::memory_order_relaxed);
        g_dev_cus[dev].store(cus, std::memory_order_release);
    }
    out->id = dev;
    out->cus = cus;
    out->lds_max = (size_t)g_dev_lds[dev].load(std::memory_order_relaxed);
    return FDBB_OK;
}

// ------------------------------------------------------------ launch table

struct Config {
    int block;
    int ppt;
    int grid_cap;
    int nt;
};

uint64_t pack(const Config &c)
{
    return (uint64_t)(uint16_t)c.block | ((uint64_t)(uint8_t)c.ppt << 16) | ((uint64_t)(c.nt ? 1 : 0) << 24) |
           ((uint64_t)(uint32_t)c.grid_cap << 32);
}

Config unpack(uint64_t v)
{
    Config c;
    c.block = (int)(v & 0xffff);
    c.ppt = (int)((v >> 16) & 0xff);
    c.nt = (int)((v >> 24) & 1);
    c.grid_cap = (int)(uint32_t)(v >> 32);
    return c;
}

std::atomic<uint64_t> g_cfg[FDBB_NUM_OPS][3][2];
std::once_flag g_cfg_once;

// The small-launch entries: calls of n <= g_small_max points take
// g_small_cfg (no entry while g_small_max is 0).  The setter stores the
// configuration before the bound and the remover clears the bound first, so
// a launch that sees a non-zero bound also sees a configuration that was
// valid for this (op, dim, dtype).
std::atomic<uint64_t> g_small_cfg[FDBB_NUM_OPS][3][2];
std::atomic<int64_t> g_small_max[FDBB_NUM_OPS][3][2];

// The library's own choice for both (the defaults below, or the installed
// table): a launch with these values may be fitted to its rows, one with
// others is a caller's and stays as it is.
std::atomic<uint64_t> g_own_cfg[FDBB_NUM_OPS][3][2];
std::atomic<uint64_t> g_own_small_cfg[FDBB_NUM_OPS][3][2];

// Beside its own small entry the library may have one for fewer points ([0],
// up to the bound), and beside its own other one one for more ([1], from the
// bound on); a bound of 0 is none.  No two shapes fit all sizes: waves of one
// point per thread that just exceed what the chip holds leave it almost empty
// for the last of them (1D cons2prim FP64, 128 x 1: 1.14 of the best at 2^20
// points), where shapes of 4 points per thread lose half below 2^17.
std::atomic<uint64_t> g_level_cfg[2][FDBB_NUM_OPS][3][2];
std::atomic<int64_t> g_level_bound[2][FDBB_NUM_OPS][3][2];

void init_configs()
{
    for (int op = 0; op < FDBB_NUM_OPS; ++op)
        for (int d = 0; d < 3; ++d)
            for (int t = 0; t < 2; ++t) {
                Config c;
                // one point per thread where a point holds many registers
                // (staged Jacobian blocks; the viscous flux's K + D*D + D
                // input and K*D output fields)
                const bool wide = (op == FDBB_OP_FLUX_JACOBIAN || op == FDBB_OP_FUSED || op == FDBB_OP_VISCOUS_FLUX);
                c.block = 256;
                c.ppt = wide ? 1 : (t == FDBB_F64 ? 2 : 4);
                c.grid_cap = 0;
                c.nt = 1;
                g_cfg[op][d][t].store(pack(c));
                g_own_cfg[op][d][t].store(pack(c));
            }
}

Config get_config(int op, int dim, int dtype)
{
    std::call_once(g_cfg_once, init_configs);
    return unpack(g_cfg[op][dim - 1][dtype].load(std::memory_order_relaxed));
}

Config get_config(int op, int dim, int dtype, int64_t n, bool *own = nullptr)
{
    const int64_t max_n = g_small_max[op][dim - 1][dtype].load(std::memory_order_acquire);
    const bool small = max_n > 0 && n <= max_n;
    const Config c = small ? unpack(g_small_cfg[op][dim - 1][dtype].load(std::memory_order_relaxed))
                           : get_config(op, dim, dtype);
    const bool ours = pack(c) == (small ? g_own_small_cfg : g_own_cfg)[op][dim - 1][dtype].load(std::memory_order_relaxed);
    if (own) *own = ours;
    if (!ours) return c;
    const int level = small ? 0 : 1;
    const int64_t bound = g_level_bound[level][op][dim - 1][dtype].load(std::memory_order_acquire);
    if (bound == 0 || (small ? n > bound : n < bound)) return c;
    return unpack(g_level_cfg[level][op][dim - 1][dtype].load(std::memory_order_relaxed));
}

// Launch configuration of the batch kernels, per storage type:
// what plans created with block == 0 (and the request server's plans) use.
// grid_per_cu 0 sizes the grid to 2048 / block workgroups per compute unit.
struct BatchConfig {
    int block;
    int ppt;
    int grid_per_cu;
    int nt;  // 0 regular, 1 nt, 2 nt + sc1
};

// [0] FP64, [1] FP32, [2] the request server's batched launches
std::atomic<uint64_t> g_batch_cfg[3] = {{0}, {0}, {0}};

uint64_t pack_batch(const BatchConfig &c)
{
    return (uint64_t)(uint16_t)c.block | ((uint64_t)(uint8_t)c.ppt << 16) | ((uint64_t)(uint8_t)c.nt << 24) |
           ((uint64_t)(uint32_t)c.grid_per_cu << 32);
}

// dtype FDBB_F64 or FDBB_F32, or 2 for the server's entry
BatchConfig get_batch_config(int dtype)
{
    const uint64_t v = g_batch_cfg[dtype == FDBB_F32 ? 1 : (dtype == 2 ? 2 : 0)].load(std::memory_order_relaxed);
    if (v == 0) return BatchConfig{256, 1, 0, 1};
    BatchConfig c;
    c.block = (int)(v & 0xffff);
    c.ppt = (int)((v >> 16) & 0xff);
    c.nt = (int)((v >> 24) & 0xff);
    c.grid_per_cu = (int)(uint32_t)(v >> 32);
    return c;
}

bool batch_config_ok(int block, int ppt, int nt)
{
    return block >= 64 && block <= kMaxBlockStaged && block % 64 == 0 &&
           (ppt == 1 || ppt == 2 || ppt == 4 || ppt == 8) && nt >= 0 && nt <= 2;
}

bool config_ok(int block, int ppt, int grid_cap, int nt)
{
    return block >= 64 && block <= 1024 && block % 64 == 0 && (ppt == 1 || ppt == 2 || ppt == 4) &&
           grid_cap >= 0 && (nt == 0 || nt == 1);
}

// ------------------------------------------------------------ validation

// Byte range of a field set: `fields` rows of stride ld, the last one n long,
// each element `unit` elements of T wide (K*K for Jacobian blocks).
struct Range {
    uintptr_t lo, hi;
    bool input;
    const void *base;
    int64_t ld;
    int task;
};

Range field_range(const void *base, int64_t ld, int64_t fields, int64_t n, int64_t unit, size_t es,
                  bool input, int task = 0)
{
    Range r;
    r.lo = (uintptr_t)base;
    r.hi = r.lo + (uintptr_t)(((fields - 1) * ld + n) * unit) * es;
    r.input = input;
    r.base = base;
    r.ld = ld;
    r.task = task;
    return r;
}

bool overlap(const Range &a, const Range &b) { return a.lo < b.hi && b.lo < a.hi; }

int check_common(int dim, double gamma, int dtype, int64_t n)
{
    if (dim < 1 || dim > 3) return fail(FDBB_EINVAL, "dim must be 1, 2 or 3");
    if (!std::isfinite(gamma) || !(gamma > 1.0)) return fail(FDBB_EINVAL, "gamma must be finite and > 1");
    if (dtype != FDBB_F64 && dtype != FDBB_F32) return fail(FDBB_EINVAL, "unknown dtype");
    if (n < 0) return fail(FDBB_EINVAL, "n must be >= 0");
    if (n >= FDBB_MAX_POINTS) return fail(FDBB_EINVAL, "n must be below 2^31 points per call");
    return FDBB_OK;
}

Gas make_gas(double gamma)
{
    Gas g;
    g.gamma = gamma;
    g.g1 = gamma - 1.0;
    g.half_g1 = 0.5 * (gamma - 1.0);
    g.inv_g1 = 1.0 / (gamma - 1.0);
    g.two_inv_g1 = 2.0 / (gamma - 1.0);
    g.quarter_g1 = 0.25 * (gamma - 1.0);
    g.inv_gamma = 1.0 / gamma;
    g.p_inf = 0.0;
    g.inv_cv = 0.0;
    g.mu = 0.0;
    g.kappa = 0.0;
    return g;
}

// Everything one launch needs, built and validated on the host.
struct Call {
    int op = 0, dim = 0, dtype = 0;
    Args a{};
    Range ranges[8];            // field sets of the call, for alias checks
    int nranges = 0;
    bool inplace_ok = false;    // K -> K transform
};

// Register one field set: checks NULL, ld and alignment.
int add_fields(Call &c, const void *base, int64_t ld, int64_t fields, int64_t unit, bool input,
               bool required, const char *name)
{
    const int64_t n = c.a.n;
    const size_t es = elem_size(c.dtype);
    if (base == nullptr) {
        if (required && n > 0) return fail(FDBB_EINVAL, std::string(name) + " must not be NULL");
        return FDBB_OK;
    }
    if (fields > 1 && ld < n) return fail(FDBB_EINVAL, std::string("ld of ") + name + " must be >= n");
    if ((uintptr_t)base % es != 0)
        return fail(FDBB_EALIGN, std::string(name) + " is not aligned to its element size");
    if (n > 0) {
        if (c.nranges >= 8) return fail(FDBB_EINVAL, "too many field sets in one call");
        c.ranges[c.nranges++] = field_range(base, fields > 1 ? ld : 0, fields, n, unit, es, input);
    }
    return FDBB_OK;
}

int check_alias(const Call &c)
{
    const Range *R = c.ranges;
    for (int i = 0; i < c.nranges; ++i)
        for (int j = i + 1; j < c.nranges; ++j) {
            if (R[i].input && R[j].input) continue;
            if (!overlap(R[i], R[j])) continue;
            const bool exact = R[i].base == R[j].base && R[i].ld == R[j].ld && R[i].input != R[j].input;
            if (exact && c.inplace_ok) continue;
            return fail(FDBB_EALIAS, "input and output field sets overlap");
        }
    return FDBB_OK;
}

int family_of(int op)
{
    switch (op) {
    case FDBB_OP_CONS2PRIM: return kFamCons2Prim;
    case FDBB_OP_PRIM2CONS: return kFamPrim2Cons;
    case FDBB_OP_EOS: return kFamEos;
    case FDBB_OP_FLUX:
    case FDBB_OP_FLUX_DIR: return kFamFlux;
    case FDBB_OP_RIEMANN: return kFamRiemann;
    case FDBB_OP_CONS2CHAR: return kFamCons2Char;
    case FDBB_OP_CHAR2CONS: return kFamChar2Cons;
    case FDBB_OP_FLUX_JACOBIAN:
    case FDBB_OP_FUSED: return kFamFused;
    case FDBB_OP_ADJOINT: return kFamAdjoint;
    case FDBB_OP_V_MAG2: return kFamVmag2;
    case FDBB_OP_EIGENVECTORS: return kFamEigen;
    case FDBB_OP_CHAR_APPLY: return kFamCharApply;
    case FDBB_OP_ROE_AVERAGE: return kFamRoe;
    case FDBB_OP_EOS_PVT: return kFamEosPvt;
    case FDBB_OP_VISCOUS_FLUX: return kFamViscous;
    default: return -1;
    }
}

const void *kernel_for(int op, int dim, int dtype, int ppt, bool nt)
{
    const int fam = family_of(op);
    switch (fam) {
    case kFamCons2Prim:
    case kFamPrim2Cons:
    case kFamEos:
    case kFamFlux:
    case kFamRiemann:
    case kFamVmag2:
    case kFamRoe:
    case kFamEosPvt:
    case kFamViscous: return kernel_pointwise(fam, dim, dtype, ppt, nt);
    case kFamCons2Char:
    case kFamChar2Cons: return kernel_char(fam, dim, dtype, ppt, nt);
    case kFamFused: return kernel_fused(dim, dtype, ppt, nt, op == FDBB_OP_FUSED);
    case kFamAdjoint: return kernel_adjoint(dim, dtype, ppt, nt);
    case kFamEigen:
    case kFamCharApply: return kernel_eigen(fam, dim, dtype, ppt, nt);
    default: return nullptr;
    }
}

bool stages_blocks(int op) { return family_of(op) == kFamFused || family_of(op) == kFamEigen; }

size_t lds_bytes(int op, int dim, int dtype, int block, int ppt)
{
    if (!stages_blocks(op)) return 0;
    // Jacobian blocks only need staging when they are written.
    const size_t K = (size_t)dim + 2;
    return (size_t)block * ppt * K * K * elem_size(dtype);
}

// Values one point writes (every output of a pointwise op).
int written_values(int op, int dim)
{
    const int K = dim + 2;
    switch (op) {
    case FDBB_OP_EOS: return 2;
    case FDBB_OP_EOS_PVT: return 3;
    case FDBB_OP_V_MAG2: return 1;
    case FDBB_OP_FLUX:
    case FDBB_OP_VISCOUS_FLUX: return K * dim;
    case FDBB_OP_RIEMANN: return 2 * dim + 1;
    default: return K;
    }
}

// How a call's output is dealt to workgroups (see Split), and what a
// workgroup writes.
struct SplitPlan {
    Split dev{1, 1, {}};
    bool blocks = false;  // K x K blocks are staged in LDS
    bool split = false;   // one set of parts per workgroup
    bool cached = false;  // the output fits in the last-level cache
    int written = 0;      // bytes one point writes in the widest set of parts
};

// The ways of dealing, timed on the same buffers (3D unless noted; time over
// that of one workgroup per tile, every part of it, at its best shape):
//   kByDirection (FP64): 0.87 at 1 000 003 points, 0.95 from 4 M to 2^24;
//     rows apart 0.88 / 0.96, so the state is read three times, not four;
//   kFieldsApart (FP32): 0.85-0.95 from 1 000 003 to 1.5 M points (by
//     direction 2-4 % slower), but only while a program's arrays together stay
//     below about 4 GB: at 2.5 M points 0.87 over one set of arrays, 0.85 over
//     4 and 1.21 over 12 in turn (whole tile 0.96, 0.97, 0.93), at 8 M 0.86
//     over one and 1.24 over 4 (0.99, 0.99); up to 512 MiB of blocks even 12
//     sets gain (0.93), beyond the whole tile is taken.  Eigenvector blocks
//     keep their split up to 6 GiB: over one, two and four sets 0.87, 0.96 and
//     0.90 at 7 M points (whole tile 1.00, 0.97, 0.91), 0.89, 0.93 and 0.99 at
//     12 M (0.98, 0.91, 0.92), 1.00, 0.99 and 1.04 at 2^24 (0.89, 0.89, 0.93);
//   1D and 2D (K*K a power of two or 9): the whole tile, a split gained
//     nothing (2D FP64 0.92 against 0.93, 2D FP32 1.02 against 1.00);
//   blocks that fit in the 256 MB last-level cache: the whole tile (200 003
//     points FP32 split 1.12, FP64 0.96).
// Spans of 131072 points: 32768 is level in FP64 (0.933 against 0.930 over 16
// buffers), 10-20 % slower in FP32; one span over the whole call reads the
// state from HBM again (2^24 FP64: 1.05).
constexpr int64_t kApartMaxBytes = (int64_t)512 << 20, kEigenApartMaxBytes = (int64_t)6 << 30;
constexpr int64_t kLastLevelBytes = (int64_t)256 << 20;
enum { kWhole = 0, kByDirection = 1, kFieldsApart = 2 };

// Only for one point per thread without a grid cap: more points per thread
// write as much per workgroup as a bounded set should, and lose by the split
// (3D FP64 Jacobian at 128 x 4 threads x points 1.14-1.17).
bool one_point(const Config &cfg) { return cfg.ppt == 1 && cfg.grid_cap == 0; }

SplitPlan split_of(const Call &c, const Config &cfg)
{
    const int D = c.dim, K = D + 2;
    const int es = (int)elem_size(c.dtype);
    SplitPlan p;
    Split &sp = p.dev;
    sp.span = (uint32_t)std::max<int64_t>(1, kSpanPoints / ((int64_t)cfg.block * cfg.ppt));
    const auto add = [&](uint32_t mask, int values) {
        sp.mask[sp.groups++] = mask;
        p.written = std::max(p.written, values * es);
    };
    int mode = D < 3 ? kWhole : c.dtype == FDBB_F64 ? kByDirection : kFieldsApart;
    const bool eigen = c.op == FDBB_OP_EIGENVECTORS;
    const int64_t block_bytes = (int64_t)(eigen ? 2 : 1) * D * K * K * es * c.a.n;
    if (c.dtype == FDBB_F32 && block_bytes > (eigen ? kEigenApartMaxBytes : kApartMaxBytes)) mode = kWhole;
    p.cached = block_bytes <= kLastLevelBytes;
    if (p.cached || !one_point(cfg)) mode = kWhole;
    p.split = mode != kWhole;
    if (c.op == FDBB_OP_EIGENVECTORS) {
        sp.groups = 0;
        p.blocks = true;
        uint32_t all = 0;
        for (int k = 0; k < 2 * D; ++k)
            if ((k & 1) ? c.a.out1 != nullptr : c.a.out0 != nullptr) all |= 1u << k;
        if (mode == kWhole) add(all, K * K * __builtin_popcount(all));
        else
            for (int k = 0; k < 2 * D; ++k)
                if (all >> k & 1u) add(1u << k, K * K);
    } else if (family_of(c.op) == kFamFused) {
        sp.groups = 0;
        p.blocks = c.a.out1 != nullptr;
        const int rows = (c.a.out0 ? K * D : 0) + (c.a.out2 ? 2 * D + 1 : 0);
        const uint32_t dirs = (1u << D) - 1u;
        if (mode == kWhole || !p.blocks) {
            add(dirs << kPartFields | dirs, rows + (p.blocks ? D * K * K : 0));
        } else if (mode == kFieldsApart) {
            if (rows) add(dirs << kPartFields, rows);
            for (int d = 0; d < D; ++d) add(1u << d, K * K);
        } else {
            for (int d = 0; d < D; ++d) add(1u << d | 1u << (kPartFields + d), K * K + (rows + D - 1) / D);
        }
    } else {
        p.written = written_values(c.op, D) * es;
    }
    return p;
}

// Output rows that start inside a cache line (packed tensors of odd length,
// offset views) split a line between every two workgroups, which usually run
// on different XCDs and each write their part of it to memory.  Longer runs
// leave fewer such lines: the pointwise ops that write a field set take at
// least 512 threads at one point each (time over the table's shape, mean over
// dims, types and packed sets of 1 to 12 M points: characteristic product
// 0.89, Roe average and adjoint 0.90, viscous flux and characteristic
// transforms 0.94); the transforms only where the table gives a thread one
// point (1D cons2char at 2 and 4 points: 1.09 and 1.28).  The streaming stores
// of the flux and the Riemann invariants carry sc1, which writes parts of
// lines through at once; in 2D and 3D regular stores, which L2 merges, are
// faster then (flux 0.77, 0.91, 0.64, 0.81 for 2D FP32, FP64, 3D FP32, FP64;
// invariants 0.87, 0.96, 0.81, 0.92; 1D 0.98 to 1.13, left alone).  Below 2^19
// points or 8 MiB of output the rows stay in cache and nothing changes (1D
// FP32 characteristic product of 600 011 points 1.08); one direction's flux
// needs 24 MiB (3D FP32: 600 011 points 1.11, 1 000 003 1.05, 2 500 009 0.89).
constexpr int64_t kLineBytes = 128;
constexpr int64_t kRaggedMin = (int64_t)1 << 19;
constexpr int64_t kRaggedBytes = (int64_t)8 << 20, kRaggedDirBytes = (int64_t)24 << 20;
constexpr int kRaggedBlock = 512;

bool ragged_rows(const Call &c)
{
    const uintptr_t starts = (uintptr_t)c.a.out0 | (uintptr_t)(c.a.ld_out0 * (int64_t)elem_size(c.dtype));
    return c.a.n >= kRaggedMin && starts % kLineBytes != 0;
}

Config fit_rows(const Call &c, Config cfg)
{
    const int64_t bytes = written_values(c.op, c.dim) * (int64_t)elem_size(c.dtype) * c.a.n;
    if (!ragged_rows(c) || bytes < (c.op == FDBB_OP_FLUX_DIR ? kRaggedDirBytes : kRaggedBytes)) return cfg;
    switch (family_of(c.op)) {
    case kFamFlux:
    case kFamRiemann:
        if (c.dim == 1) return cfg;
        cfg.nt = 0;
        break;
    case kFamCons2Char:
    case kFamChar2Cons:
        if (cfg.ppt != 1) return cfg;
        break;
    case kFamAdjoint:
    case kFamCharApply:
    case kFamRoe:
    case kFamViscous: break;
    default: return cfg;
    }
    cfg.block = std::max(cfg.block, kRaggedBlock);
    cfg.ppt = 1;
    cfg.grid_cap = 0;
    return cfg;
}

// Waves that may be resident on a compute unit.  A wave writes as many rows
// as its op has output fields, far apart in memory, so every resident wave
// adds that many open DRAM rows; past about 57 KB of output in flight per
// compute unit (900 B per lane) more waves only make the rows of different
// fields displace each other.  3D flux FP64 (120 B written per point) at
// 12 000 017 points: 8 waves 301 us, 16 waves 316, unlimited (32) 353; 2D
// flux FP64 (64 B): 10 waves 178, unlimited 200; 3D Riemann invariants FP64
// (56 B): 12-16 waves 1 % off the best, unlimited 6 %.  Below 8 waves the
// loads of the next waves no longer cover the latency (3D flux FP64 at 6
// waves: 310 us; 1D flux FP32 at 8: 2.4 times slower), and ops that write
// 32 B or less keep every wave.
//
// Kernels that stage blocks take 1536 B per lane of a split set: 4 waves of
// 256-thread workgroups in 3D FP64 (fused pass at 12 000 017 points: 4 waves
// 0.95 of the unsplit time, 8 waves 1.01, 12 waves 1.05), 12 in FP32 (0.85;
// 8 waves 0.89, 24 waves 0.99).  A whole tile at one point per thread takes
// 3072 B in 2D FP64 (fused pass 8 waves 0.93, 16 waves 1.00), 2048 B in 1D
// FP64 (16 waves 0.95, 24 waves 0.97, 12 waves 1.01) and 6208 B in FP32 (3D
// beyond 512 MiB: 16 waves 0.93-1.00); blocks that stay in the last-level
// cache keep every wave.
//
// Rows are bounded where a call writes 192 MiB or more, three quarters of the
// last-level cache: smaller calls drain into it, and few waves then cost more
// at the ramp and the tail than they save (time with the bound over that
// without, 3D flux FP64: 300 007 points 1.03, 1.5 M 1.08, 1.9 M 1.03, 2.5 M
// 0.91; 2D viscous flux FP64: 300 007 1.06, 1.2 M 1.02, 3 M 0.97).  Rows that
// start inside cache lines are bounded from 48 MiB (2D viscous flux FP64, 1 M
// and 2.5 M points 0.96 and 0.92, 600 011 1.02; 3D flux FP64 600 011 0.94).
// More than one point per thread has fewer and heavier waves to begin with and
// keeps them all: 2D viscous flux FP32 at 4 points each took 1.4 times as long
// with the bound, 1D cons2prim FP64 of 1 000 003 points at 4 each 1.16 times.
constexpr int kMaxWaves = 32, kMinWaves = 8;
constexpr int kWrittenPerLane = 900;
constexpr int64_t kBoundedBytes = (int64_t)192 << 20, kRaggedBoundedBytes = (int64_t)48 << 20;

int resident_waves(const SplitPlan &p, const Call &c, const Config &cfg)
{
    if (!one_point(cfg)) return kMaxWaves;
    if (p.blocks) {
        int per_lane = 1536;
        if (!p.split) {
            if (p.cached) return kMaxWaves;
            per_lane = c.dtype == FDBB_F32 ? 6208 : c.dim == 1 ? 2048 : 3072;
        }
        return std::min(kMaxWaves, std::max(1, per_lane / p.written));
    }
    if (p.written * c.a.n < (ragged_rows(c) ? kRaggedBoundedBytes : kBoundedBytes)) return kMaxWaves;
    const int waves = std::max(kMinWaves, (kWrittenPerLane + p.written / 2) / p.written);
    return waves >= kMaxWaves - 4 ? kMaxWaves : waves;
}

// Dynamic LDS that keeps at most about `waves` waves in workgroups of
// `block` threads resident on a compute unit (0: no limit): the kernel need
// not touch it, it takes the space of the workgroups that should wait.
// Allocations are made in steps of 1280 bytes.
size_t residency_lds(int waves, int block, bool blocks, const DeviceInfo &dev)
{
    if (waves >= kMaxWaves) return 0;
    const int groups = std::max(1, (waves * 64 + (blocks ? 0 : block / 2)) / block);
    return dev.lds_max / groups / 1280 * 1280;
}

// Kernels whose dynamic-LDS limit has been raised on a device, as an
// open-addressed set of (kernel address | device << 56) keys.  The limit is
// raised once, to the device maximum, the first time a kernel needs more
// than the default 64 KB; later launches only look the key up (no lock, no
// runtime call).  Two threads may both raise it for the same kernel the
// first time; the call is idempotent.
constexpr int kAttrSlots = 4096;
std::atomic<uintptr_t> g_attr_done[kAttrSlots];

int set_lds_attr(const void *fn, size_t lds, const DeviceInfo &dev)
{
    if (lds <= 65536) return FDBB_OK;
    if (lds > dev.lds_max) return fail(FDBB_EINVAL, "launch configuration needs more LDS than a workgroup may use");
    const uintptr_t key = (uintptr_t)fn | ((uintptr_t)(dev.id + 1) << 56);
    size_t h = (size_t)((key >> 4) * 0x9E3779B97F4A7C15ull) % kAttrSlots;
    for (int probe = 0; probe < kAttrSlots; ++probe, h = (h + 1) % kAttrSlots) {
        uintptr_t v = g_attr_done[h].load(std::memory_order_acquire);
        if (v == key) return FDBB_OK;
        if (v != 0) continue;
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dev.lds_max);
        if (e != hipSuccess) return fail_hip(e, "hipFuncSetAttribute");
        uintptr_t expected = 0;
        if (g_attr_done[h].compare_exchange_strong(expected, key, std::memory_order_acq_rel)) return FDBB_OK;
        if (expected == key) return FDBB_OK;
        // another kernel took this slot meanwhile: keep probing
    }
    return FDBB_OK;  // table full (more kernels than exist): the limit is raised anyway
}

// `alone`: the call may count on the whole chip.  Few resident waves are
// right for one launch's streams; a launch that shares the chip with others'
// would only give them its place (a saturated server's p99 3.95 -> 3.65 ms).
int launch(Call &c, void *stream, bool alone = true)
{
    if (c.a.n == 0) return FDBB_OK;
    int rc = check_alias(c);
    if (rc) return rc;

    bool own = false;
    Config cfg = get_config(c.op, c.dim, c.dtype, c.a.n, &own);
    if (own) cfg = fit_rows(c, cfg);
    const void *fn = kernel_for(c.op, c.dim, c.dtype, cfg.ppt, cfg.nt != 0);
    if (!fn) return fail(FDBB_EINVAL, "no kernel for this configuration");
    DeviceInfo dev;
    rc = device_info(&dev);
    if (rc) return rc;
    const int64_t tile_pts = (int64_t)cfg.block * cfg.ppt;
    int64_t ntiles = (c.a.n + tile_pts - 1) / tile_pts;
    SplitPlan sp = split_of(c, cfg);
    size_t lds = sp.blocks ? lds_bytes(c.op, c.dim, c.dtype, cfg.block, cfg.ppt) : 0;
    if (alone) lds = std::max(lds, residency_lds(resident_waves(sp, c, cfg), cfg.block, sp.blocks, dev));
    rc = set_lds_attr(fn, lds, dev);
    if (rc) return rc;

    int64_t grid = ntiles * sp.dev.groups;
    if (cfg.grid_cap > 0 && grid > cfg.grid_cap) grid = cfg.grid_cap;
    // keep a dispatch below 2^31 work-items (the grid-dimension bound HIP
    // reports on this device); the kernels loop over tiles, so a capped grid
    // still covers every point
    const int64_t max_grid = 0x7fffffffLL / cfg.block;
    if (grid > max_grid) grid = max_grid;
    void *args[] = {&c.a, &ntiles, &sp.dev};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3((unsigned)cfg.block), args, lds,
                                   (hipStream_t)stream);
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return FDBB_OK;
}

int begin(Call &c, int op, int dim, double gamma, int dtype, int64_t n)
{
    int rc = check_common(dim, gamma, dtype, n);
    if (rc) return rc;
    c.op = op;
    c.dim = dim;
    c.dtype = dtype;
    c.a.n = n;
    c.a.gas = make_gas(gamma);
    g_last_error.clear();
    return FDBB_OK;
}

// Whether in0 and in1 are views of the same K rows, shifted by so few points
// that what one side read is still cached when the other asks for it: the
// lines of that distance, a quarter of the last-level cache at most.  Roe
// average of 8 M points, 3D FP64, time over that of unrelated sides' path:
// 0.57 at 1 cell, 0.72 at 1000, 0.85 at 1.5 M (60 MB), 1.04 at 7 M (280 MB).
constexpr int64_t kNearBytes = (int64_t)64 << 20;

bool near_views(const fdbb_task &t, int K)
{
    if (t.ld_in0 != t.ld_in1) return false;
    const uintptr_t l = (uintptr_t)t.in0, r = (uintptr_t)t.in1;
    const int64_t shift = (int64_t)(l < r ? r - l : l - r);  // bytes
    return shift < t.n * (int64_t)elem_size(t.dtype) && shift * K <= kNearBytes;
}

// Fills c for any op from the task-style argument list; shared by the
// single-call entry points and the batch plans.  `mode` selects R (1) or L
// (0) for the characteristic products.
int build_call(Call &c, const fdbb_task &t, int mode = 0)
{
    int rc = begin(c, t.op, t.dim, t.gamma, t.dtype, t.n);
    if (rc) return rc;
    const int D = t.dim, K = D + 2;
    Args &a = c.a;
    a.dir = 0;
    switch (t.op) {
    case FDBB_OP_CONS2PRIM:
    case FDBB_OP_PRIM2CONS:
    case FDBB_OP_CONS2CHAR:
    case FDBB_OP_CHAR2CONS: {
        if (t.op == FDBB_OP_CONS2CHAR || t.op == FDBB_OP_CHAR2CONS) {
            if (t.dir < 0 || t.dir >= D) return fail(FDBB_EINVAL, "dir out of range");
            a.dir = t.dir;
        }
        c.inplace_ok = true;
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "input"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, K, 1, false, true, "output"))) return rc;
        if (t.in0 == t.out0 && t.ld_in0 == t.ld_out0 &&
            (t.op == FDBB_OP_CONS2PRIM || t.op == FDBB_OP_PRIM2CONS))
            a.flags |= kFlagInPlace;
        break;
    }
    case FDBB_OP_EOS:
        if (!t.out0 && !t.out1 && t.n > 0) return fail(FDBB_EINVAL, "p and c must not both be NULL");
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.out1 = t.out1;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, 0, 1, 1, false, false, "p"))) return rc;
        if ((rc = add_fields(c, t.out1, 0, 1, 1, false, false, "c"))) return rc;
        break;
    case FDBB_OP_FLUX:
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, (int64_t)K * D, 1, false, true, "F"))) return rc;
        break;
    case FDBB_OP_FLUX_DIR:
        if (t.dir < 0 || t.dir >= D) return fail(FDBB_EINVAL, "dir out of range");
        a.dir = t.dir;
        a.flags |= kFlagOneDir;
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, K, 1, false, true, "F_dir"))) return rc;
        break;
    case FDBB_OP_EIGENVECTORS:
        if (!t.out0 && !t.out1 && t.n > 0) return fail(FDBB_EINVAL, "L and R must not both be NULL");
        a.in0 = t.in0, a.ld_in0 = t.ld_in0;
        a.out0 = t.out0, a.ld_out0 = t.ld_out0, a.out1 = t.out1, a.ld_out1 = t.ld_out1;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, D, (int64_t)K * K, false, false, "L"))) return rc;
        if ((rc = add_fields(c, t.out1, t.ld_out1, D, (int64_t)K * K, false, false, "R"))) return rc;
        break;
    case FDBB_OP_CHAR_APPLY:
        if (t.dir < 0 || t.dir >= D) return fail(FDBB_EINVAL, "dir out of range");
        if (mode != 0 && mode != 1) return fail(FDBB_EINVAL, "mode must be 0 (L) or 1 (R)");
        a.dir = t.dir;
        if (mode == 1) a.flags |= kFlagRight;
        c.inplace_ok = true;
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.in1 = t.in1, a.ld_in1 = t.ld_in1;
        a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.in1, t.ld_in1, K, 1, true, true, "X"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, K, 1, false, true, "Y"))) return rc;
        break;
    case FDBB_OP_EOS_PVT:
        if (!t.out0 && !t.out1 && !t.out2 && t.n > 0) return fail(FDBB_EINVAL, "p, c and T must not all be NULL");
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.out1 = t.out1, a.out2 = t.out2;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, 0, 1, 1, false, false, "p"))) return rc;
        if ((rc = add_fields(c, t.out1, 0, 1, 1, false, false, "c"))) return rc;
        if ((rc = add_fields(c, t.out2, 0, 1, 1, false, false, "T"))) return rc;
        break;
    case FDBB_OP_ROE_AVERAGE:
        c.inplace_ok = true;
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.in1 = t.in1, a.ld_in1 = t.ld_in1;
        a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if (near_views(t, K)) a.flags |= kFlagShared;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "UL"))) return rc;
        if ((rc = add_fields(c, t.in1, t.ld_in1, K, 1, true, true, "UR"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, K, 1, false, true, "Uh"))) return rc;
        break;
    case FDBB_OP_V_MAG2:
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, D + 1, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, 0, 1, 1, false, true, "y"))) return rc;
        break;
    case FDBB_OP_RIEMANN:
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, 2 * D + 1, 1, false, true, "R"))) return rc;
        break;
    case FDBB_OP_FLUX_JACOBIAN:
        // The Jacobian blocks travel in out1 of the fused kernel.
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.out1 = t.out0, a.ld_out1 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, D, (int64_t)K * K, false, true, "A"))) return rc;
        break;
    case FDBB_OP_FUSED:
        if (!t.out0 && !t.out1 && !t.out2 && t.n > 0) return fail(FDBB_EINVAL, "F, A and R must not all be NULL");
        a.in0 = t.in0, a.ld_in0 = t.ld_in0;
        a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        a.out1 = t.out1, a.ld_out1 = t.ld_out1;
        a.out2 = t.out2, a.ld_out2 = t.ld_out2;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, (int64_t)K * D, 1, false, false, "F"))) return rc;
        if ((rc = add_fields(c, t.out1, t.ld_out1, D, (int64_t)K * K, false, false, "A"))) return rc;
        if ((rc = add_fields(c, t.out2, t.ld_out2, 2 * D + 1, 1, false, false, "R"))) return rc;
        break;
    case FDBB_OP_ADJOINT:
        if (t.dir < -1 || t.dir >= D) return fail(FDBB_EINVAL, "dir out of range");
        a.dir = t.dir;
        a.in0 = t.in0, a.ld_in0 = t.ld_in0, a.in1 = t.in1, a.ld_in1 = t.ld_in1;
        a.out0 = t.out0, a.ld_out0 = t.ld_out0;
        if ((rc = add_fields(c, t.in0, t.ld_in0, K, 1, true, true, "U"))) return rc;
        if ((rc = add_fields(c, t.in1, t.ld_in1, t.dir < 0 ? (int64_t)K * D : K, 1, true, true, "Fbar")))
            return rc;
        if ((rc = add_fields(c, t.out0, t.ld_out0, K, 1, false, true, "Ubar"))) return rc;
        break;
    case FDBB_OP_VISCOUS_FLUX:
        return fail(FDBB_EINVAL, "the viscous flux needs its gradients and coefficients: call fdbb_viscous_flux");
    default: return fail(FDBB_EINVAL, "unknown op");
    }
    return FDBB_OK;
}

// Ops a batch plan can run: everything the general batch kernel dispatches.
// The eigenvector blocks and characteristic products have kernels of their
// own, and the general EOS needs parameters a task does not carry.
bool batchable(int op)
{
    return op >= 0 && op < FDBB_NUM_OPS && op != FDBB_OP_EIGENVECTORS && op != FDBB_OP_CHAR_APPLY &&
           op != FDBB_OP_EOS_PVT && op != FDBB_OP_VISCOUS_FLUX;
}

fdbb_task make_task(int op, int dim, int dir, double gamma, int dtype, int64_t n)
{
    fdbb_task t;
    std::memset(&t, 0, sizeof(t));
    t.op = op;
    t.dim = dim;
    t.dir = dir;
    t.gamma = gamma;
    t.dtype = dtype;
    t.n = n;
    return t;
}

int run(const fdbb_task &t, void *stream, int mode = 0)
{
    Call c;
    int rc = build_call(c, t, mode);
    if (rc) return rc;
    return launch(c, stream);
}

}  // namespace

namespace fdbb {

// fdbb_task_run of a valid task beside launches on other streams.
int task_run_among_others(const fdbb_task &task, void *stream)
{
    Call c;
    int rc = build_call(c, task);
    return rc ? rc : launch(c, stream, false);
}

}  // namespace fdbb

// ================================================================ C ABI

extern "C" {

int fdbb_cons2prim(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *V, int64_t ldV,
                   int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_CONS2PRIM, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = V, t.ld_out0 = ldV;
    return run(t, stream);
}

int fdbb_prim2cons(int dim, double gamma, int dtype, const void *V, int64_t ldV, void *U, int64_t ldU,
                   int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_PRIM2CONS, dim, 0, gamma, dtype, n);
    t.in0 = V, t.ld_in0 = ldV, t.out0 = U, t.ld_out0 = ldU;
    return run(t, stream);
}

int fdbb_velocity_magnitude2(int dim, int dtype, const void *U, int64_t ldU, void *y, int64_t n, void *stream)
{
    // gamma does not enter |v|^2; any valid value passes validation
    fdbb_task t = make_task(FDBB_OP_V_MAG2, dim, 0, 1.4, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = y;
    return run(t, stream);
}

int fdbb_eos(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *p, void *c, int64_t n,
             void *stream)
{
    fdbb_task t = make_task(FDBB_OP_EOS, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = p, t.out1 = c;
    return run(t, stream);
}

int fdbb_flux(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *F, int64_t ldF, int64_t n,
              void *stream)
{
    fdbb_task t = make_task(FDBB_OP_FLUX, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = F, t.ld_out0 = ldF;
    return run(t, stream);
}

int fdbb_flux_direction(int dim, int dir, double gamma, int dtype, const void *U, int64_t ldU, void *Fd,
                        int64_t ldFd, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_FLUX_DIR, dim, dir, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = Fd, t.ld_out0 = ldFd;
    return run(t, stream);
}

int fdbb_flux_jacobian(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *A, int64_t ldA,
                       int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_FLUX_JACOBIAN, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = A, t.ld_out0 = ldA;
    return run(t, stream);
}

int fdbb_riemann_invariants(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *R,
                            int64_t ldR, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_RIEMANN, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = R, t.ld_out0 = ldR;
    return run(t, stream);
}

int fdbb_cons2char(int dim, int dir, double gamma, int dtype, const void *U, int64_t ldU, void *W,
                   int64_t ldW, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_CONS2CHAR, dim, dir, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = W, t.ld_out0 = ldW;
    return run(t, stream);
}

int fdbb_char2cons(int dim, int dir, double gamma, int dtype, const void *W, int64_t ldW, void *U,
                   int64_t ldU, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_CHAR2CONS, dim, dir, gamma, dtype, n);
    t.in0 = W, t.ld_in0 = ldW, t.out0 = U, t.ld_out0 = ldU;
    return run(t, stream);
}

int fdbb_euler_fused(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *F, int64_t ldF,
                     void *A, int64_t ldA, void *R, int64_t ldR, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_FUSED, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU;
    t.out0 = F, t.ld_out0 = ldF;
    t.out1 = A, t.ld_out1 = ldA;
    t.out2 = R, t.ld_out2 = ldR;
    return run(t, stream);
}

int fdbb_flux_adjoint(int dim, int dir, double gamma, int dtype, const void *U, int64_t ldU,
                      const void *Fbar, int64_t ldFbar, void *Ubar, int64_t ldUbar, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_ADJOINT, dim, dir, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.in1 = Fbar, t.ld_in1 = ldFbar, t.out0 = Ubar, t.ld_out0 = ldUbar;
    return run(t, stream);
}

int fdbb_eigenvectors(int dim, double gamma, int dtype, const void *U, int64_t ldU, void *L, int64_t ldL,
                      void *R, int64_t ldR, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_EIGENVECTORS, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = L, t.ld_out0 = ldL, t.out1 = R, t.ld_out1 = ldR;
    return run(t, stream);
}

int fdbb_char_apply(int dim, int dir, int mode, double gamma, int dtype, const void *U, int64_t ldU,
                    const void *X, int64_t ldX, void *Y, int64_t ldY, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_CHAR_APPLY, dim, dir, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.in1 = X, t.ld_in1 = ldX, t.out0 = Y, t.ld_out0 = ldY;
    return run(t, stream, mode);
}

int fdbb_roe_average(int dim, double gamma, int dtype, const void *UL, int64_t ldUL, const void *UR,
                     int64_t ldUR, void *Uh, int64_t ldUh, int64_t n, void *stream)
{
    fdbb_task t = make_task(FDBB_OP_ROE_AVERAGE, dim, 0, gamma, dtype, n);
    t.in0 = UL, t.ld_in0 = ldUL, t.in1 = UR, t.ld_in1 = ldUR, t.out0 = Uh, t.ld_out0 = ldUh;
    return run(t, stream);
}

int fdbb_eos_pvt(int dim, int eos, const double *params, int dtype, const void *U, int64_t ldU, void *p,
                 void *c, void *T, int64_t n, void *stream)
{
    g_last_error.clear();
    if (!params) return fail(FDBB_EINVAL, "params must not be NULL");
    double gamma = 0.0, p_inf = 0.0, cv = 0.0;
    if (eos == FDBB_EOS_PERFECT_GAS) {
        const double cp = params[0];
        cv = params[1];
        if (!std::isfinite(cp) || !std::isfinite(cv) || !(cv > 0.0) || !(cp > cv))
            return fail(FDBB_EINVAL, "perfect gas needs c_p > c_v > 0");
        gamma = cp / cv;
    } else if (eos == FDBB_EOS_STIFFENED_GAS) {
        gamma = params[0];
        p_inf = params[1];
        cv = params[2];
        if (!std::isfinite(p_inf) || !(p_inf >= 0.0) || !std::isfinite(cv) || !(cv > 0.0))
            return fail(FDBB_EINVAL, "stiffened gas needs p_inf >= 0 and c_v > 0");
    } else {
        return fail(FDBB_EINVAL, "unknown EOS id");
    }
    fdbb_task t = make_task(FDBB_OP_EOS_PVT, dim, 0, gamma, dtype, n);
    t.in0 = U, t.ld_in0 = ldU, t.out0 = p, t.out1 = c, t.out2 = T;
    Call call;
    int rc = build_call(call, t);
    if (rc) return rc;
    call.a.gas.p_inf = p_inf;
    call.a.gas.inv_cv = 1.0 / cv;
    return launch(call, stream);
}

int fdbb_viscous_flux(int dim, double mu, double kappa, int dtype, const void *U, int64_t ldU, const void *G,
                      int64_t ldG, const void *gradT, int64_t ldGT, void *Fv, int64_t ldFv, int64_t n,
                      void *stream)
{
    Call c;
    // gamma does not enter the viscous flux; any valid value passes the checks
    int rc = begin(c, FDBB_OP_VISCOUS_FLUX, dim, 2.0, dtype, n);
    if (rc) return rc;
    if (!std::isfinite(mu) || !(mu >= 0.0) || !std::isfinite(kappa) || !(kappa >= 0.0))
        return fail(FDBB_EINVAL, "mu and kappa must be finite and >= 0");
    const int64_t D = dim, K = D + 2;
    Args &a = c.a;
    a.in0 = U, a.ld_in0 = ldU, a.in1 = G, a.ld_in1 = ldG, a.in2 = gradT, a.ld_in2 = ldGT;
    a.out0 = Fv, a.ld_out0 = ldFv;
    a.gas.mu = mu;
    a.gas.kappa = kappa;
    if ((rc = add_fields(c, U, ldU, K, 1, true, true, "U"))) return rc;
    if ((rc = add_fields(c, G, ldG, D * D, 1, true, true, "G"))) return rc;
    if ((rc = add_fields(c, gradT, ldGT, D, 1, true, true, "gradT"))) return rc;
    if ((rc = add_fields(c, Fv, ldFv, K * D, 1, false, true, "Fv"))) return rc;
    return launch(c, stream);
}

int fdbb_task_check(const fdbb_task *task)
{
    if (!task) return fail(FDBB_EINVAL, "task must not be NULL");
    if (task->op == FDBB_OP_EOS_PVT) return fail(FDBB_EINVAL, "the general EOS needs its parameters: call fdbb_eos_pvt");
    Call c;
    int rc = build_call(c, *task);
    if (!rc) rc = check_alias(c);
    return rc;
}

int fdbb_task_run(const fdbb_task *task, void *stream)
{
    if (!task) return fail(FDBB_EINVAL, "task must not be NULL");
    if (task->op == FDBB_OP_EOS_PVT) return fail(FDBB_EINVAL, "the general EOS needs its parameters: call fdbb_eos_pvt");
    return run(*task, stream);
}

int fdbb_set_launch_config(int op, int dim, int dtype, int block, int ppt, int grid_cap, int nontemporal)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    if (!config_ok(block, ppt, grid_cap, nontemporal)) return fail(FDBB_EINVAL, "invalid launch configuration");
    if (stages_blocks(op) && block > kMaxBlockStaged)
        return fail(FDBB_EINVAL, "kernels that stage K x K blocks take at most 256 threads per workgroup");
    std::call_once(g_cfg_once, init_configs);
    Config c{block, ppt, grid_cap, nontemporal};
    g_cfg[op][dim - 1][dtype].store(pack(c));
    return FDBB_OK;
}

int fdbb_get_launch_config(int op, int dim, int dtype, int *block, int *ppt, int *grid_cap, int *nontemporal)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    const Config c = get_config(op, dim, dtype);
    if (block) *block = c.block;
    if (ppt) *ppt = c.ppt;
    if (grid_cap) *grid_cap = c.grid_cap;
    if (nontemporal) *nontemporal = c.nt;
    return FDBB_OK;
}

int fdbb_set_small_launch_config(int op, int dim, int dtype, int64_t max_n, int block, int ppt, int grid_cap,
                                 int nontemporal)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    if (max_n < 0) return fail(FDBB_EINVAL, "max_n must not be negative");
    if (max_n == 0) {
        g_small_max[op][dim - 1][dtype].store(0, std::memory_order_release);
        return FDBB_OK;
    }
    if (!config_ok(block, ppt, grid_cap, nontemporal)) return fail(FDBB_EINVAL, "invalid launch configuration");
    if (stages_blocks(op) && block > kMaxBlockStaged)
        return fail(FDBB_EINVAL, "kernels that stage K x K blocks take at most 256 threads per workgroup");
    // clear the bound while the configuration changes, then publish both
    g_small_max[op][dim - 1][dtype].store(0, std::memory_order_release);
    g_small_cfg[op][dim - 1][dtype].store(pack(Config{block, ppt, grid_cap, nontemporal}), std::memory_order_relaxed);
    g_small_max[op][dim - 1][dtype].store(max_n, std::memory_order_release);
    return FDBB_OK;
}

int fdbb_install_launch_config(int op, int dim, int dtype, int level, int64_t bound, int block, int ppt, int grid_cap,
                               int nontemporal)
{
    if (level < 0 || level > 3) return fail(FDBB_EINVAL, "level must be 0 to 3");
    const uint64_t packed = pack(Config{block, ppt, grid_cap, nontemporal});
    if (level == 1 || level == 2) {
        const int rc = level == 2 ? fdbb_set_launch_config(op, dim, dtype, block, ppt, grid_cap, nontemporal)
                                  : fdbb_set_small_launch_config(op, dim, dtype, bound, block, ppt, grid_cap, nontemporal);
        if (rc == FDBB_OK && (level == 2 || bound > 0))
            (level == 2 ? g_own_cfg : g_own_small_cfg)[op][dim - 1][dtype].store(packed, std::memory_order_relaxed);
        return rc;
    }
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    if (bound < 0) return fail(FDBB_EINVAL, "bound must not be negative");
    if (bound > 0 && !config_ok(block, ppt, grid_cap, nontemporal)) return fail(FDBB_EINVAL, "invalid launch configuration");
    if (bound > 0 && stages_blocks(op) && block > kMaxBlockStaged)
        return fail(FDBB_EINVAL, "kernels that stage K x K blocks take at most 256 threads per workgroup");
    // clear the bound while the configuration changes, then publish both
    std::atomic<int64_t> &b = g_level_bound[level == 0 ? 0 : 1][op][dim - 1][dtype];
    b.store(0, std::memory_order_release);
    g_level_cfg[level == 0 ? 0 : 1][op][dim - 1][dtype].store(packed, std::memory_order_relaxed);
    b.store(bound, std::memory_order_release);
    return FDBB_OK;
}

int fdbb_get_small_launch_config(int op, int dim, int dtype, int64_t *max_n, int *block, int *ppt, int *grid_cap,
                                 int *nontemporal)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    const int64_t m = g_small_max[op][dim - 1][dtype].load(std::memory_order_acquire);
    const Config c = m > 0 ? unpack(g_small_cfg[op][dim - 1][dtype].load(std::memory_order_relaxed))
                           : get_config(op, dim, dtype);
    if (max_n) *max_n = m;
    if (block) *block = c.block;
    if (ppt) *ppt = c.ppt;
    if (grid_cap) *grid_cap = c.grid_cap;
    if (nontemporal) *nontemporal = c.nt;
    return FDBB_OK;
}

int fdbb_launch_config_for(int op, int dim, int dtype, int64_t n, int *block, int *ppt, int *grid_cap,
                           int *nontemporal)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32))
        return fail(FDBB_EINVAL, "unknown op, dim or dtype");
    if (n < 0) return fail(FDBB_EINVAL, "n must not be negative");
    const Config c = get_config(op, dim, dtype, n);
    if (block) *block = c.block;
    if (ppt) *ppt = c.ppt;
    if (grid_cap) *grid_cap = c.grid_cap;
    if (nontemporal) *nontemporal = c.nt;
    return FDBB_OK;
}

int fdbb_kernel_info(int op, int dim, int dtype, int ppt, int nontemporal, int *vgprs, int *scratch_bytes)
{
    if (op < 0 || op >= FDBB_NUM_OPS || dim < 1 || dim > 3 || (dtype != FDBB_F64 && dtype != FDBB_F32) ||
        !(ppt == 1 || ppt == 2 || ppt == 4) || (nontemporal != 0 && nontemporal != 1))
        return fail(FDBB_EINVAL, "unknown op, dim, dtype, ppt or store mode");
    const void *fn = kernel_for(op, dim, dtype, ppt, nontemporal != 0);
    if (!fn) return fail(FDBB_EINVAL, "no kernel for this configuration");
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, fn);
    if (e != hipSuccess) return fail_hip(e, "hipFuncGetAttributes");
    if (vgprs) *vgprs = attr.numRegs;
    if (scratch_bytes) *scratch_bytes = (int)attr.localSizeBytes;
    return FDBB_OK;
}

const char *fdbb_status_string(int status)
{
    switch (status) {
    case FDBB_OK: return "ok";
    case FDBB_EINVAL: return "invalid argument";
    case FDBB_EALIGN: return "misaligned pointer";
    case FDBB_EALIAS: return "input and output overlap";
    case FDBB_EHIP: return "HIP runtime error";
    case FDBB_ENOMEM: return "out of memory";
    default: return "unknown status";
    }
}

const char *fdbb_last_error(void) { return g_last_error.c_str(); }

int fdbb_version(void) { return 400; }

}  // extern "C"

// ================================================================ batches

// Layout of a task table, on the device and in its host staging copy:
// [header: ntasks, ntiles (int64)][tile prefix sums, cap + 1 int64][pad to
// 64 B][cap TaskDev].
static size_t table_task_offset(int cap) { return ((2 + (size_t)cap + 1) * sizeof(int64_t) + 63) & ~(size_t)63; }
static size_t table_bytes(int cap) { return table_task_offset(cap) + (size_t)cap * sizeof(TaskDev); }
static int64_t *table_header(unsigned char *base) { return reinterpret_cast<int64_t *>(base); }
static int64_t *table_prefix(unsigned char *base) { return reinterpret_cast<int64_t *>(base) + 2; }
static TaskDev *table_tasks(unsigned char *base, int cap) { return reinterpret_cast<TaskDev *>(base + table_task_offset(cap)); }

// What a batch launches with.
struct BatchLaunch {
    const void *kernel = nullptr;
    int block = 256;
    int ppt = 1;
    int nt = 1;
    int grid = 0;
    size_t lds = 0;      // dynamic LDS: what the list stages, or more to bound residency
    bool parts = false;  // a tile's parts are dealt to several units

    bool operator==(const BatchLaunch &o) const
    {
        return kernel == o.kernel && block == o.block && grid == o.grid && lds == o.lds;
    }
};

// A task list as the host knows it.
struct TaskList {
    int ntasks = 0;
    int64_t points = 0;
    int64_t tiles = 0;  // of the creation shape
    BatchLaunch launch;  // its own
};

// The plan's table: the layout above with its prefix sums in tiles of the
// creation shape, which the general launch reads, behind a second header and
// second prefix sums (cap + 1) in units of the current list's own launch.
struct fdbb_batch_plan {
    int device = 0;
    int capacity = 0;
    bool installed = false;     // block == 0 at creation: the installed configurations
    bool general_only = false;  // a list was uploaded inside a capture (see fdbb_batch_plan_update)
    BatchLaunch base;           // as created; base.lds is the staging a task list may need
    size_t general_lds = 0;     // what the general launch takes for it
    TaskList cur;               // the last one uploaded
    BatchLaunch captured;       // what `exec` launches with
    unsigned char *dev = nullptr;   // task table, capacity `capacity`
    unsigned char *host = nullptr;  // pinned staging copy of the same layout
    size_t bytes = 0;
    hipEvent_t uploaded = nullptr;  // the last upload has left the staging copy
    hipGraphExec_t exec = nullptr;  // the first list's own launch (none for a plan created empty)

    size_t units_bytes() const { return ((2 + (size_t)capacity + 1) * sizeof(int64_t) + 63) & ~(size_t)63; }
    int64_t *unit_header(unsigned char *t) const { return reinterpret_cast<int64_t *>(t); }
    int64_t *unit_prefix(unsigned char *t) const { return reinterpret_cast<int64_t *>(t) + 2; }
    unsigned char *table(unsigned char *t) const { return t + units_bytes(); }
};

namespace {

// Whether a task writes K x K blocks.
bool writes_blocks(const fdbb_task &t) { return t.op == FDBB_OP_FLUX_JACOBIAN || (t.op == FDBB_OP_FUSED && t.out1); }

// LDS that the tasks' blocks are staged in at this shape.
size_t staged_lds(const fdbb_task *tasks, int ntasks, int block, int ppt)
{
    size_t lds = 0;
    for (int b = 0; b < ntasks; ++b)
        if (writes_blocks(tasks[b])) lds = std::max(lds, lds_bytes(tasks[b].op, tasks[b].dim, tasks[b].dtype, block, ppt));
    return lds;
}

// LDS of the general kernel in a caller's shape: where it stages blocks at one
// point per thread, with regular or nt stores, at most 8 waves are resident.
// Its registers allow 12, which the streams of a 2D tile displace one another
// at: lists of fused passes at 256 threads, 8 workgroups per compute unit, 2D
// FP32 6 M points 212 us against 190, 2D FP64 600 K points 48 against 43.
size_t general_lds(const BatchLaunch &l, size_t staged, const DeviceInfo &dev)
{
    return staged && l.ppt == 1 && l.nt != 2 ? std::max(staged, residency_lds(8, l.block, true, dev)) : staged;
}

// Sets of parts a block-writing 3D task's tiles are dealt in when they are
// dealt apart, as split_of deals a single call's.
int task_groups(const fdbb_task &t)
{
    const bool rows = t.op == FDBB_OP_FUSED && (t.out0 || t.out2);
    return t.dtype == FDBB_F32 && rows ? t.dim + 1 : t.dim;
}

// Kernel and shape of a task list (valid tasks), timed against one workgroup
// per tile and the general kernel, on the same buffers.
//
// A plan of explicit shape launches the general kernel in it: the rest is for
// the installed configurations, whose shapes it was timed in (at 64 x 4
// threads x points, a 3D FP64 list of 6 M points dealt apart took 1.51 times as
// long as the general kernel, at 128 x 1 with 4 workgroups per compute unit an
// FP32 one of 1.3 M points 1.53 times).  Parts and bounds also need one point
// per thread and a grid that leaves the order of units to the hardware.
//
// A list of block-writing tasks of one dim and storage type takes the fused
// batch kernel (time over the general kernel's at its best shape):
//   3D FP64, parts by direction, 8 waves: 0.89 at 14 M points in 96 tasks,
//     0.92 at 3 M in 40 (whole tile, 4 waves: 0.95 and 0.94; parts at 4
//     waves 1.09, 6 waves 1.1, unlimited 0.97); from 32 GiB of blocks the
//     whole tile at 4 waves wins (72.8 M in 512 tasks 0.97, by parts 1.01;
//     55 M 0.96 and 0.96; 40 M 0.96 and 0.88);
//   3D FP32, parts without a bound up to 512 MiB of blocks, as in a single
//     call: 0.64 at 1.5 M points; beyond the whole tile at 16 waves: 0.79 at 3
//     M, 0.94 at 10 M, 0.93 at 8.7 M over three sets of arrays in turn (parts
//     0.72, 1.00, 1.02), 25 M 0.95;
//   2D whole tile: FP64 8 waves 0.95 (unlimited 1.03), FP32 0.72; 1D 0.78
//     and 0.53 without a bound (16 waves 0.78 and 0.76);
//   lists that fit in the last-level cache: the whole tile, no bound and, in
//     2D and 3D, regular stores (3D FP64 200 K points 0.93, streaming 1.02;
//     1D 900 K 0.92 streaming, 1.03 regular).
// Any other list takes the general kernel at 128 threads and, unless its grid
// is smaller, a workgroup per tile: one point per thread where it stages 2D or
// 3D blocks (48 mixed requests of 733 MB: 0.75 of the fused shape's time; 2
// points 0.81), else two (1D and 3D flux FP64 0.92 and 0.84; 1 point 1.3 and
// 0.90).
constexpr int64_t kListApartMaxBytes = (int64_t)32 << 30;

BatchLaunch pick_launch(const fdbb_task *tasks, int ntasks, const BatchLaunch &base, bool installed,
                        const DeviceInfo &dev)
{
    BatchLaunch l = base;
    l.lds = staged_lds(tasks, ntasks, l.block, l.ppt);
    if (!installed) {
        l.lds = general_lds(l, l.lds, dev);
        return l;
    }
    const fdbb_task *first = nullptr;
    bool uniform = true;
    int rows = 0;
    int64_t points = 0;
    for (int b = 0; b < ntasks; ++b) {
        const fdbb_task &t = tasks[b];
        if (t.n == 0) continue;
        if (!first) first = &t;
        uniform = writes_blocks(t) && t.dim == first->dim && t.dtype == first->dtype;
        if (!uniform) break;
        if (t.op == FDBB_OP_FUSED)
            rows = std::max(rows, (t.out0 ? (t.dim + 2) * t.dim : 0) + (t.out2 ? 2 * t.dim + 1 : 0));
        points += t.n;
    }
    if (!first) return l;
    if (uniform) {
        const int D = first->dim, KK = (D + 2) * (D + 2), es = (int)elem_size(first->dtype);
        const void *k = kernel_batch_fused(D, first->dtype, base.ppt, base.nt);
        if (k) {
            const bool f64 = first->dtype == FDBB_F64;
            const int64_t block_bytes = (int64_t)D * KK * es * points;
            const bool cached = block_bytes + (int64_t)rows * es * points <= kLastLevelBytes;
            const bool dealt = l.ppt == 1 && l.grid >= dev.cus * 64;
            l.parts = D == 3 && dealt && !cached && block_bytes <= (f64 ? kListApartMaxBytes : kApartMaxBytes);
            const int written = es * l.ppt * (!l.parts ? rows + D * KK : f64 ? KK + (rows + D - 1) / D : KK);
            int per_lane = 0;  // bytes that the resident waves write per lane, 0: no bound
            if (l.parts) per_lane = f64 ? 2200 : 0;
            else if (!cached && D > 1 && dealt) per_lane = f64 ? 3072 : 6208;
            const int waves = per_lane ? std::max(1, std::min(kMaxWaves, per_lane / written)) : kMaxWaves;
            if (cached && D > 1) l.nt = 0, k = kernel_batch_fused(D, first->dtype, l.ppt, l.nt);
            l.kernel = k;
            l.lds = std::max(lds_bytes(FDBB_OP_FLUX_JACOBIAN, D, first->dtype, l.block, l.ppt),
                             residency_lds(waves, l.block, true, dev));
            return l;
        }
    }
    bool staged = false;
    for (int b = 0; b < ntasks; ++b) staged = staged || (writes_blocks(tasks[b]) && tasks[b].dim > 1);
    l.block = 128, l.ppt = staged ? 1 : 2, l.nt = staged ? 2 : 1;
    l.grid = dev.cus * 64;
    l.kernel = kernel_batch(l.ppt, l.nt);
    l.lds = staged_lds(tasks, ntasks, l.block, l.ppt);
    return l;
}

// The units of the launch `l` over `ntasks` tasks: fills the second header
// and prefix sums and each task's part of them, and cuts the grid to the
// units there are.
void fill_units(int ntasks, BatchLaunch &l, int64_t *hdr, int64_t *pre, TaskDev *td, const fdbb_task *tasks)
{
    const int64_t tile_pts = (int64_t)l.block * l.ppt;
    int64_t units = 0;
    for (int b = 0; b < ntasks; ++b) {
        td[b].groups = l.parts ? task_groups(tasks[b]) : 1;
        td[b].first_unit = pre[b] = units;
        units += (tasks[b].n + tile_pts - 1) / tile_pts * td[b].groups;
    }
    pre[ntasks] = units;
    hdr[0] = ntasks;
    hdr[1] = units;
    l.grid = (int)std::max<int64_t>(1, std::min<int64_t>(l.grid, units));
}

// What filling a task table found.
struct TableInfo {
    size_t lds = 0;      // dynamic LDS the tasks' Jacobian staging needs
    int64_t tiles = 0;
    int64_t points = 0;
};

// Validate `tasks` (each as its single-call entry point would, then every
// pair of tasks for overlapping outputs) and write the table for tiles of
// block * ppt points into `host` (layout above, capacity `cap`).  `all`
// must have room for 8 * ntasks ranges.  Uses no heap memory of its own.
int fill_table(const fdbb_task *tasks, int ntasks, int cap, int block, int ppt, unsigned char *host, Range *all,
               TableInfo *info)
{
    if (ntasks > 0 && !tasks) return fail(FDBB_EINVAL, "tasks must not be NULL");
    int64_t *hdr = table_header(host);
    int64_t *pre = table_prefix(host);
    TaskDev *td = table_tasks(host, cap);
    const int64_t tile_pts = (int64_t)block * ppt;
    size_t nall = 0;
    TableInfo r;
    for (int b = 0; b < ntasks; ++b) {
        if (!batchable(tasks[b].op))
            return fail(FDBB_EINVAL, "task " + std::to_string(b) + ": op not available in batches");
        Call c;
        int rc = build_call(c, tasks[b]);
        if (rc) return fail(rc, "task " + std::to_string(b) + ": " + g_last_error);
        rc = check_alias(c);
        if (rc) return fail(rc, "task " + std::to_string(b) + ": " + g_last_error);
        if (writes_blocks(tasks[b])) r.lds = std::max(r.lds, lds_bytes(tasks[b].op, tasks[b].dim, tasks[b].dtype, block, ppt));
        for (int k = 0; k < c.nranges; ++k) {
            all[nall] = c.ranges[k];
            all[nall].task = b;
            ++nall;
        }
        pre[b] = r.tiles;
        r.tiles += (tasks[b].n + tile_pts - 1) / tile_pts;
        r.points += tasks[b].n;
        td[b].a = c.a;
        td[b].op = tasks[b].op;
        td[b].dim = tasks[b].dim;
        td[b].dtype = tasks[b].dtype;
        td[b].groups = 1;
        td[b].first_unit = pre[b];
    }
    // Across tasks: no output may overlap another task's input or output.
    std::sort(all, all + nall, [](const Range &x, const Range &y) { return x.lo < y.lo; });
    for (size_t i = 0; i < nall; ++i) {
        for (size_t j = i + 1; j < nall && all[j].lo < all[i].hi; ++j) {
            if (all[i].task == all[j].task) continue;
            if (all[i].input && all[j].input) continue;
            return fail(FDBB_EALIAS, "tasks " + std::to_string(all[i].task) + " and " +
                                         std::to_string(all[j].task) + " overlap");
        }
    }
    pre[ntasks] = r.tiles;
    hdr[0] = ntasks;
    hdr[1] = r.tiles;
    *info = r;
    return FDBB_OK;
}

// Validate tasks and fill the plan's pinned staging copy.
int stage_tasks(fdbb_batch_plan *p, const fdbb_task *tasks, int ntasks, TaskList *next)
{
    if (ntasks < 0 || ntasks > p->capacity) return fail(FDBB_EINVAL, "ntasks exceeds the plan capacity");
    if (ntasks > 0 && !tasks) return fail(FDBB_EINVAL, "tasks must not be NULL");
    DeviceInfo dev;
    int rc = device_info(&dev);
    if (rc) return rc;
    // Fill a private copy first, so that a rejected list neither waits for
    // nor disturbs an upload still reading the staging copy.
    const size_t used = p->units_bytes() + table_task_offset(p->capacity) + (size_t)ntasks * sizeof(TaskDev);
    std::vector<unsigned char> tmp(used);
    std::vector<Range> all((size_t)ntasks * 8);
    TableInfo info;
    unsigned char *table = p->table(tmp.data());
    rc = fill_table(tasks, ntasks, p->capacity, p->base.block, p->base.ppt, table, all.data(), &info);
    if (rc) return rc;
    if (info.lds > p->base.lds) return fail(FDBB_EINVAL, "tasks need more LDS than the plan was created with");
    BatchLaunch l = pick_launch(tasks, ntasks, p->base, p->installed, dev);
    if ((rc = set_lds_attr(l.kernel, l.lds, dev))) return rc;
    fill_units(ntasks, l, p->unit_header(tmp.data()), p->unit_prefix(tmp.data()), table_tasks(table, p->capacity), tasks);
    // The previous upload must have consumed the staging copy.
    if (p->uploaded) {
        hipError_t e = hipEventSynchronize(p->uploaded);
        if (e != hipSuccess) return fail_hip(e, "hipEventSynchronize");
    }
    std::memcpy(p->host, tmp.data(), used);
    *next = TaskList{ntasks, info.points, info.tiles, l};
    return FDBB_OK;
}

// Whether `s` is being captured.  The query fails on the default stream while
// another stream is: `s` itself is not, then.
bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// Uploads the staged list, which becomes the plan's once the copy is queued:
// after a copy that failed, the table is still the one that the list before
// launches over.
int upload(fdbb_batch_plan *p, const TaskList &next, hipStream_t s)
{
    // A captured upload runs when its graph is replayed: until then the device
    // table is another list's, so such a plan keeps to the general launch.
    const bool captured = capturing(s);
    // header, prefix sums and the tasks in use (not the whole capacity)
    const size_t used = p->units_bytes() + table_task_offset(p->capacity) + (size_t)next.ntasks * sizeof(TaskDev);
    hipError_t e = hipMemcpyAsync(p->dev, p->host, used, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return fail_hip(e, "hipMemcpyAsync");
    p->cur = next;
    if (captured) p->general_only = true;
    e = hipEventRecord(p->uploaded, s);
    if (e != hipSuccess) {
        // nothing else keeps the next list from the staging copy
        (void)hipStreamSynchronize(s);
        return fail_hip(e, "hipEventRecord");
    }
    return FDBB_OK;
}

// The general launch of p's table in the creation shape.  It takes any list
// that the plan accepts, so its dynamic LDS is what any of them may stage: a
// launch that is captured, or that runs before a captured upload does, may
// find another list in the table than the current one.
int launch_general(fdbb_batch_plan *p, hipStream_t s)
{
    unsigned char *t = p->table(p->dev);
    const TaskDev *tasks = table_tasks(t, p->capacity);
    const int64_t *prefix = table_prefix(t);
    const int64_t *header = table_header(t);
    void *args[] = {&tasks, &prefix, &header};
    const BatchLaunch &l = p->base;
    hipError_t e = hipLaunchKernel(l.kernel, dim3((unsigned)l.grid), dim3((unsigned)l.block), args, p->general_lds, s);
    if (e != hipSuccess) return fail_hip(e, "batch kernel launch");
    return FDBB_OK;
}

// The current list's own launch.
int launch_list(fdbb_batch_plan *p, hipStream_t s)
{
    const TaskDev *tasks = table_tasks(p->table(p->dev), p->capacity);
    const int64_t *prefix = p->unit_prefix(p->dev);
    const int64_t *header = p->unit_header(p->dev);
    void *args[] = {&tasks, &prefix, &header};
    const BatchLaunch &l = p->cur.launch;
    hipError_t e = hipLaunchKernel(l.kernel, dim3((unsigned)l.grid), dim3((unsigned)l.block), args, l.lds, s);
    if (e != hipSuccess) return fail_hip(e, "batch kernel launch");
    return FDBB_OK;
}

// Captures what `launch` puts on a stream of its own and instantiates it.
template <typename F>
int capture(hipGraphExec_t *exec, F launch)
{
    hipStream_t cs = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
    if (e != hipSuccess) return fail_hip(e, "hipStreamCreateWithFlags");
    hipGraph_t graph = nullptr;
    int rc = FDBB_OK;
    e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        rc = launch(cs);
        hipError_t e2 = hipStreamEndCapture(cs, &graph);
        if (rc == FDBB_OK && e2 != hipSuccess) rc = fail_hip(e2, "hipStreamEndCapture");
    } else {
        rc = fail_hip(e, "hipStreamBeginCapture");
    }
    (void)hipStreamDestroy(cs);
    if (rc == FDBB_OK) {
        e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) rc = fail_hip(e, "hipGraphInstantiate");
    }
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
}

void free_plan(fdbb_batch_plan *p)
{
    if (!p) return;
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->uploaded) (void)hipEventDestroy(p->uploaded);
    if (p->dev) (void)hipFree(p->dev);
    if (p->host) (void)hipHostFree(p->host);
    delete p;
}

}  // namespace

extern "C" {

int fdbb_batch_plan_create(const fdbb_task *tasks, int ntasks, int capacity, int block, int ppt, int grid,
                           int nontemporal, fdbb_batch_plan **plan)
{
    g_last_error.clear();
    if (!plan) return fail(FDBB_EINVAL, "plan must not be NULL");
    *plan = nullptr;
    if (capacity < 1 || capacity < ntasks) return fail(FDBB_EINVAL, "capacity must be >= max(1, ntasks)");
    if (ntasks > 0 && !tasks) return fail(FDBB_EINVAL, "tasks must not be NULL");
    int grid_per_cu = 0;
    const bool installed = block == 0;
    if (installed) {
        // the installed configuration of the first task's storage type
        const BatchConfig bc = get_batch_config(ntasks > 0 ? tasks[0].dtype : FDBB_F64);
        block = bc.block, ppt = bc.ppt, nontemporal = bc.nt, grid_per_cu = bc.grid_per_cu, grid = 0;
    }
    if (!batch_config_ok(block, ppt, nontemporal) || grid < 0)
        return fail(FDBB_EINVAL, "invalid launch configuration (batches take 64..256 threads per workgroup in "
                                 "multiples of 64, 1, 2, 4 or 8 points per thread, store mode 0, 1 or 2)");
    // Argument checks of every task come before any HIP call.
    for (int b = 0; b < ntasks; ++b) {
        if (!batchable(tasks[b].op))
            return fail(FDBB_EINVAL, "task " + std::to_string(b) + ": op not available in batches");
        Call c;
        int rc = build_call(c, tasks[b]);
        if (!rc) rc = check_alias(c);
        if (rc) return fail(rc, "task " + std::to_string(b) + ": " + g_last_error);
    }
    DeviceInfo dev;
    int rc = device_info(&dev);
    if (rc) return rc;

    fdbb_batch_plan *p = new fdbb_batch_plan();
    p->capacity = capacity;
    p->installed = installed;
    p->base.block = block;
    p->base.ppt = ppt;
    p->base.nt = nontemporal;
    p->base.kernel = kernel_batch(ppt, nontemporal);
    p->base.grid = grid > 0 ? grid : dev.cus * (grid_per_cu > 0 ? grid_per_cu : std::max(1, 2048 / block));
    (void)hipGetDevice(&p->device);
    // LDS for the largest Jacobian staging among the first task list; a plan
    // created empty reserves enough for any task (3D FP64 blocks).
    p->base.lds = ntasks == 0 ? lds_bytes(FDBB_OP_FLUX_JACOBIAN, 3, FDBB_F64, block, ppt)
                              : staged_lds(tasks, ntasks, block, ppt);
    p->general_lds = general_lds(p->base, p->base.lds, dev);
    if ((rc = set_lds_attr(p->base.kernel, p->general_lds, dev))) {
        free_plan(p);
        return rc;
    }
    p->bytes = p->units_bytes() + table_bytes(capacity);
    hipError_t e = hipMalloc((void **)&p->dev, p->bytes);
    if (e != hipSuccess) {
        free_plan(p);
        return fail_hip(e, "hipMalloc");
    }
    e = hipHostMalloc((void **)&p->host, p->bytes, hipHostMallocDefault);
    if (e != hipSuccess) {
        free_plan(p);
        return fail_hip(e, "hipHostMalloc");
    }
    std::memset(p->host, 0, p->bytes);
    e = hipEventCreateWithFlags(&p->uploaded, hipEventDisableTiming);
    if (e != hipSuccess) {
        free_plan(p);
        return fail_hip(e, "hipEventCreate");
    }
    TaskList first;
    if ((rc = stage_tasks(p, tasks, ntasks, &first))) {
        const std::string msg = g_last_error;
        free_plan(p);
        return fail(rc, msg);
    }
    e = hipMemcpy(p->dev, p->host, p->bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        free_plan(p);
        return fail_hip(e, "hipMemcpy");
    }
    p->cur = first;
    // Capture the list's own launch: it is replayed for every list that wants
    // the same one (only the device table that the kernel reads changes).
    if (ntasks > 0) {
        rc = capture(&p->exec, [&](hipStream_t cs) { return launch_list(p, cs); });
        p->captured = p->cur.launch;
    }
    if (rc) {
        const std::string msg = g_last_error;
        free_plan(p);
        return fail(rc, msg);
    }
    *plan = p;
    return FDBB_OK;
}

int fdbb_batch_plan_update(fdbb_batch_plan *plan, const fdbb_task *tasks, int ntasks, void *stream)
{
    g_last_error.clear();
    if (!plan) return fail(FDBB_EINVAL, "plan must not be NULL");
    TaskList next;
    int rc = stage_tasks(plan, tasks, ntasks, &next);
    return rc ? rc : upload(plan, next, (hipStream_t)stream);
}

int fdbb_batch_exec(fdbb_batch_plan *plan, void *stream, int use_graph)
{
    g_last_error.clear();
    if (!plan) return fail(FDBB_EINVAL, "plan must not be NULL");
    // The list's own launch fits this list only.  A launch that is captured
    // now, over an empty list too, may be replayed over a later list and is
    // the general one, launched directly: a graph launch on a stream that is
    // being captured runs at once and leaves nothing in the capture.
    if (plan->general_only || capturing((hipStream_t)stream)) return launch_general(plan, (hipStream_t)stream);
    if (plan->cur.tiles == 0) return FDBB_OK;
    if (!use_graph || !plan->exec || !(plan->cur.launch == plan->captured)) return launch_list(plan, (hipStream_t)stream);
    hipError_t e = hipGraphLaunch(plan->exec, (hipStream_t)stream);
    return e == hipSuccess ? FDBB_OK : fail_hip(e, "hipGraphLaunch");
}

int fdbb_set_batch_config(int dtype, int block, int ppt, int grid_per_cu, int nontemporal)
{
    g_last_error.clear();
    if (dtype != FDBB_F64 && dtype != FDBB_F32) return fail(FDBB_EINVAL, "unknown dtype");
    if (!batch_config_ok(block, ppt, nontemporal) || grid_per_cu < 0 || grid_per_cu > 1024)
        return fail(FDBB_EINVAL, "invalid batch configuration");
    // a plan of this configuration must be able to stage 3D Jacobian blocks
    if (lds_bytes(FDBB_OP_FLUX_JACOBIAN, 3, dtype, block, ppt) > 160 * 1024)
        return fail(FDBB_EINVAL, "batch configuration needs more LDS than a workgroup may use");
    g_batch_cfg[dtype == FDBB_F32 ? 1 : 0].store(pack_batch(BatchConfig{block, ppt, grid_per_cu, nontemporal}));
    return FDBB_OK;
}

int fdbb_set_server_batch_config(int block, int ppt, int grid_per_cu, int nontemporal)
{
    g_last_error.clear();
    if (block == 0) {
        g_batch_cfg[2].store(0);
        return FDBB_OK;
    }
    if (!batch_config_ok(block, ppt, nontemporal) || grid_per_cu < 0 || grid_per_cu > 1024)
        return fail(FDBB_EINVAL, "invalid batch configuration");
    if (lds_bytes(FDBB_OP_FLUX_JACOBIAN, 3, FDBB_F64, block, ppt) > 160 * 1024)
        return fail(FDBB_EINVAL, "batch configuration needs more LDS than a workgroup may use");
    g_batch_cfg[2].store(pack_batch(BatchConfig{block, ppt, grid_per_cu, nontemporal}));
    return FDBB_OK;
}

int fdbb_get_server_batch_config(int *block, int *ppt, int *grid_per_cu, int *nontemporal)
{
    const uint64_t v = g_batch_cfg[2].load(std::memory_order_relaxed);
    const BatchConfig c = v ? get_batch_config(2) : get_batch_config(FDBB_F64);
    if (block) *block = c.block;
    if (ppt) *ppt = c.ppt;
    if (grid_per_cu) *grid_per_cu = c.grid_per_cu;
    if (nontemporal) *nontemporal = c.nt;
    return FDBB_OK;
}

int fdbb_get_batch_config(int dtype, int *block, int *ppt, int *grid_per_cu, int *nontemporal)
{
    if (dtype != FDBB_F64 && dtype != FDBB_F32) return fail(FDBB_EINVAL, "unknown dtype");
    const BatchConfig c = get_batch_config(dtype);
    if (block) *block = c.block;
    if (ppt) *ppt = c.ppt;
    if (grid_per_cu) *grid_per_cu = c.grid_per_cu;
    if (nontemporal) *nontemporal = c.nt;
    return FDBB_OK;
}

int fdbb_batch_plan_config(const fdbb_batch_plan *plan, int *block, int *ppt, int *grid, int *nontemporal)
{
    if (!plan) return fail(FDBB_EINVAL, "plan must not be NULL");
    if (block) *block = plan->base.block;
    if (ppt) *ppt = plan->base.ppt;
    if (grid) *grid = plan->base.grid;
    if (nontemporal) *nontemporal = plan->base.nt;
    return FDBB_OK;
}

int fdbb_batch_plan_info(const fdbb_batch_plan *plan, int64_t *points, int64_t *tiles)
{
    if (!plan) return fail(FDBB_EINVAL, "plan must not be NULL");
    if (points) *points = plan->cur.points;
    if (tiles) *tiles = plan->cur.tiles;
    return FDBB_OK;
}

int fdbb_batch_plan_destroy(fdbb_batch_plan *plan)
{
    free_plan(plan);
    return FDBB_OK;
}

int fdbb_batch_run_noalloc(const fdbb_task *tasks, int ntasks, int block, int ppt, int grid, int nontemporal,
                           void *stream)
{
    g_last_error.clear();
    if (ntasks < 0 || ntasks > FDBB_NOALLOC_MAX_TASKS)
        return fail(FDBB_EINVAL, "the allocation-free batch takes 0 to " + std::to_string(FDBB_NOALLOC_MAX_TASKS) +
                                     " tasks, got " + std::to_string(ntasks));
    if (ntasks > 0 && !tasks) return fail(FDBB_EINVAL, "tasks must not be NULL");
    int grid_per_cu = 0;
    const bool installed = block == 0;
    if (installed) {
        const BatchConfig bc = get_batch_config(ntasks > 0 ? tasks[0].dtype : FDBB_F64);
        block = bc.block, ppt = bc.ppt, nontemporal = bc.nt, grid_per_cu = bc.grid_per_cu, grid = 0;
    }
    if (!batch_config_ok(block, ppt, nontemporal) || grid < 0)
        return fail(FDBB_EINVAL, "invalid launch configuration (batches take 64..256 threads per workgroup in "
                                 "multiples of 64, 1, 2, 4 or 8 points per thread, store mode 0, 1 or 2)");
    DeviceInfo dev;
    int rc = device_info(&dev);
    if (rc) return rc;
    // Host staging of the table and the range list of the overlap check:
    // static, so this call uses no heap; the lock makes concurrent callers
    // take turns over them.
    static std::mutex staging_mutex;
    alignas(64) static unsigned char staging[kNoAllocBytes];
    static Range ranges[8 * (size_t)kNoAllocMaxTasks];
    std::lock_guard<std::mutex> lock(staging_mutex);
    TableInfo info;
    rc = fill_table(tasks, ntasks, kNoAllocMaxTasks, block, ppt, staging, ranges, &info);
    if (rc) return rc;
    if (info.tiles == 0) return FDBB_OK;
    void *table = nullptr;
    const int se = batch_scratch(&table);
    if (se) return fail_hip((hipError_t)se, "hipGetSymbolAddress of the batch task table");
    BatchLaunch l;
    l.block = block, l.ppt = ppt, l.nt = nontemporal;
    l.kernel = kernel_batch(ppt, nontemporal);
    l.lds = info.lds;
    l.grid = grid > 0 ? grid : dev.cus * (grid_per_cu > 0 ? grid_per_cu : std::max(1, 2048 / block));
    if (!l.kernel) return fail(FDBB_EINVAL, "no batch kernel for this configuration");
    if ((rc = set_lds_attr(l.kernel, l.lds, dev))) return rc;
    if (!capturing((hipStream_t)stream)) {
        l = pick_launch(tasks, ntasks, l, installed, dev);
        if ((rc = set_lds_attr(l.kernel, l.lds, dev))) return rc;
    }
    fill_units(ntasks, l, table_header(staging), table_prefix(staging), table_tasks(staging, kNoAllocMaxTasks), tasks);
    // From pageable host memory the copy completes before the call returns,
    // so the staging array is free again once it does; it is ordered on
    // `stream` before the launch that reads the table.
    const size_t used = table_task_offset(kNoAllocMaxTasks) + (size_t)ntasks * sizeof(TaskDev);
    hipError_t e = hipMemcpyAsync(table, staging, used, hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e != hipSuccess) return fail_hip(e, "hipMemcpyAsync");
    unsigned char *base = static_cast<unsigned char *>(table);
    const TaskDev *dtasks = table_tasks(base, kNoAllocMaxTasks);
    const int64_t *prefix = table_prefix(base);
    const int64_t *header = table_header(base);
    void *args[] = {&dtasks, &prefix, &header};
    e = hipLaunchKernel(l.kernel, dim3((unsigned)l.grid), dim3((unsigned)l.block), args, l.lds, (hipStream_t)stream);
    if (e != hipSuccess) return fail_hip(e, "batch kernel launch");
    return FDBB_OK;
}

}  // extern "C"
