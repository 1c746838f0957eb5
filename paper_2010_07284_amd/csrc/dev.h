// dev.h -- device helpers shared by the kernels on packed masks: operand and
// descriptor access, lane shifts, the units of batched launches.  Included by
// the .hip files, each of which gets its own internal copy.
#pragma once
#include "kernels.h"

namespace vlg {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ uint32_t fdiv(uint32_t n, uint32_t mul, uint32_t shift) {
    return (uint32_t)(((uint64_t)__umulhi(n, mul) + n) >> shift);
}

// Pointers read from descriptors in memory have no known address space and
// would be accessed with flat instructions, which also count against the LDS
// wait counter; every mask, label and image access therefore goes through a
// global-qualified pointer.
#define VLG_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ VLG_GLOBAL T *glb(T *p) {
    return (VLG_GLOBAL T *)p;
}
template <typename T>
__device__ __forceinline__ const VLG_GLOBAL T *glb(const T *p) {
    return (const VLG_GLOBAL T *)p;
}
// Constant address space: for tables that no kernel writes while it runs
// (the per-image descriptors of a batched launch).  A wave-uniform index into
// them becomes a scalar load whose result stays in scalar registers.
#define VLG_CONST __attribute__((address_space(4)))

__device__ __forceinline__ uint64_t ldm(const MRef &r, int64_t i) {
    return (r.p ? glb(r.p)[i] : 0ull) ^ r.inv;
}

__device__ __forceinline__ bool is_last_col(const Geo &g, int64_t i) {
    uint32_t row = fdiv((uint32_t)i, g.wpr_mul, g.wpr_shift);
    return (uint32_t)i - row * (uint32_t)g.wpr == (uint32_t)(g.wpr - 1);
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

// Workgroups are dispatched to the 8 XCDs in turn (workgroup i to XCD
// i mod 8), and each XCD has an L2 of its own.  The work item of workgroup b
// of n: each XCD takes a contiguous range of items, so that neighbouring
// tiles, which share the cache lines of their mask words, meet in one L2
// instead of each line being fetched by several.  A bijection of [0, n).
__device__ __forceinline__ int xcd_contiguous(int b, int n) {
    constexpr int X = 8;
    const int per = n / X, rem = n % X, x = b % X, k = b / X;
    return x * per + (x < rem ? x : rem) + k;
}

int grid_for(int64_t n, int per_block, int cap) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}
// A launch whose operands add up to more than the last-level cache (256 MB
// Infinity Cache) cannot leave them cached for the next launch, so it reads
// them with the non-temporal hint (a connective over 265 MB masks went from
// 59% to over 80% of HBM peak with it); smaller launches read normally, since
// the next step of a schedule usually reads their operands again.
constexpr int64_t kStreamBytes = 256ll << 20;
template <bool NT, typename T>
__device__ __forceinline__ T ld_hint(const VLG_GLOBAL T *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// ------------------------------------------------------------------ batches
// workgroups of a persistent batched launch
int persistent_grid(const BatchArgs &a, int64_t total) {
    return grid_for(total, 1, valid_batch_grid(a.grid_cap) ? a.grid_cap : kBatchGridDefault);
}

// image of global unit u: the largest i with prefix[i] <= u.  Called by whole
// waves: 64 candidates per step (a bisection by one lane is seven dependent
// loads for 128 images, about a microsecond of every launch).
__device__ __forceinline__ int find_img(const int64_t *prefix, int n, int64_t u) {
    int lo = 0;
    for (int len = n; len > 1;) {
        const int step = (len + 63) >> 6, at = (int)(threadIdx.x & 63) * step;
        const uint64_t le = __ballot(at < len && glb(prefix)[lo + (at < len ? at : 0)] <= u);
        const int k = (le ? 63 - __builtin_clzll(le) : 0) * step;
        lo += k;
        len = step < len - k ? step : len - k;
    }
    return lo;
}

// A workgroup of a persistent batch kernel takes a contiguous range of the
// launch's global units, finds the image of its first unit by search
// and then only steps forward (units of one image are consecutive).  Kernels
// copy the image's descriptor into registers per unit: read through a
// reference into memory, its fields would be reloaded after every LDS store
// or atomic (a generic pointer may alias LDS).
struct UnitRange {
    const int64_t *prefix;
    int64_t begin, end, next;
    int ii;
    __device__ UnitRange(const int64_t *p, int n) : prefix(p) {
        const int64_t total = p[n];
        begin = total * blockIdx.x / gridDim.x;
        end = total * (blockIdx.x + 1) / gridDim.x;
        ii = begin < end ? find_img(p, n, begin) : 0;
        next = begin < end ? p[ii + 1] : 0;
    }
    __device__ __forceinline__ int img(int64_t u) {
        while (u >= next) next = prefix[++ii + 1];
        return ii;
    }
};

__device__ __forceinline__ uint64_t *bptr(const BImg &d, int32_t slot) {
    if (slot == -1) return nullptr;
    if (slot <= -2) return glb(d.outs)[-2 - slot];
    return (uint64_t *)(d.ws + (uint64_t)slot * d.mask_bytes);
}

__device__ __forceinline__ MRef bref(const BImg &d, const BRef &r) {
    MRef m;
    m.p = bptr(d, r.slot);
    m.inv = r.inv ? ~0ull : 0ull;
    return m;
}

__device__ __forceinline__ int lds_ld(int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Value of v in the previous lane of the wave (DPP wave shift right by one;
// lane 0 receives 0).
__device__ __forceinline__ int lane_prev(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, false);
}
// Value of v in the next lane of the wave (DPP wave shift left by one; lane
// 63 receives 0).
__device__ __forceinline__ int lane_next(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ uint64_t lane_prev64(uint64_t v) {
    return (uint64_t)(uint32_t)lane_prev((int)(uint32_t)v) | ((uint64_t)(uint32_t)lane_prev((int)(v >> 32)) << 32);
}
__device__ __forceinline__ uint64_t lane_next64(uint64_t v) {
    return (uint64_t)(uint32_t)lane_next((int)(uint32_t)v) | ((uint64_t)(uint32_t)lane_next((int)(v >> 32)) << 32);
}
// Raise the give-up flag of a launch, a word of the host (one store per wave).
// Called by every lane of the wave.
__device__ __forceinline__ void guard_report(const LoopGuard &gd, bool ok) {
    const uint64_t bad = __ballot(!ok);
    if (bad && lane_id() == __builtin_ctzll(bad) && gd.status)
        __hip_atomic_store(glb(gd.status), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Cross-lane handoff through LDS inside one wave: every lane's LDS writes
// before this point are complete (and visible to the other lanes) before any
// lane's LDS reads after it.  The workgroup-scope fences order the accesses
// for the compiler and wait for the outstanding LDS operations; the wave
// barrier keeps the lanes together.
__device__ __forceinline__ void wave_lds_handoff() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// The descriptor of image ii (wave-uniform) through scalar loads: the table
// is written before the launch and only read while it runs.
__device__ __forceinline__ BImg load_bimg(const BImg *imgs, int ii) {
    static_assert(sizeof(BImg) % 4 == 0, "descriptor copied as 32-bit words");
    const VLG_CONST uint32_t *p = (const VLG_CONST uint32_t *)(imgs + __builtin_amdgcn_readfirstlane(ii));
    BImg r;
    uint32_t *q = (uint32_t *)&r;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(BImg) / 4); k++) q[k] = p[k];
    return r;
}

// d: the descriptor of unit u_'s image, reloaded only when the image changes
#define VLG_BATCH_LOOP(A)                          \
    UnitRange ur_((A).prefix, (A).n);                  \
    int cur_ = -1;                                     \
    BImg dcur_;                                        \
    for (int64_t u_ = ur_.begin; u_ < ur_.end; u_++)
#define VLG_BATCH_IMG(A)                           \
    const int ii = ur_.img(u_);                        \
    if (ii != cur_) {                                  \
        dcur_ = load_bimg((A).imgs, ii);                \
        cur_ = ii;                                     \
    }                                                  \
    const BImg &d = dcur_;

}  // namespace
}  // namespace vlg
