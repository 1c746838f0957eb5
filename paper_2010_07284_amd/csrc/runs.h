// runs.h -- union-find over the runs of blocks of a mask: what the 2-D
// labelling (ccl.hip) and the volume labelling (vol.hip) share.  A lane holds
// a row of 64 blocks as 64-bit masks; horizontally connected blocks form runs.
#pragma once
#include "dev.h"

namespace vlg {
namespace {

__device__ __forceinline__ uint64_t below(int s) { return (1ull << s) - 1; }            // bits 0..s-1, s < 64
__device__ __forceinline__ uint64_t upto(int s) { return ~0ull >> (63 - s); }           // bits 0..s
// start of the run that holds block l (a set bit of the row)
__device__ __forceinline__ int run_of(uint64_t starts, int l) { return 63 - __builtin_clzll((starts & upto(l)) | 1ull); }

// Even bits of w into e, odd bits into o (an unshuffle of each half).
__device__ __forceinline__ uint32_t unshuffle32(uint32_t h) {
    uint32_t t;
    t = (h ^ (h >> 1)) & 0x22222222u; h ^= t ^ (t << 1);
    t = (h ^ (h >> 2)) & 0x0C0C0C0Cu; h ^= t ^ (t << 2);
    t = (h ^ (h >> 4)) & 0x00F000F0u; h ^= t ^ (t << 4);
    t = (h ^ (h >> 8)) & 0x0000FF00u; h ^= t ^ (t << 8);
    return h;
}
__device__ __forceinline__ void split_even_odd(uint64_t w, uint32_t &e, uint32_t &o) {
    const uint32_t lo = unshuffle32((uint32_t)w), hi = unshuffle32((uint32_t)(w >> 32));
    e = (lo & 0xFFFFu) | (hi << 16);
    o = (lo >> 16) | (hi & 0xFFFF0000u);
}
__device__ __forceinline__ uint32_t even_bits32(uint32_t x) {
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t even_bits(uint64_t w) {
    return even_bits32((uint32_t)w) | (even_bits32((uint32_t)(w >> 32)) << 16);
}
// Each bit of x twice: the pixel columns of 32 blocks.
__device__ __forceinline__ uint32_t twice16(uint32_t x) {
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    x = (x | (x << 1)) & 0x55555555u;
    return x | (x << 1);
}
__device__ __forceinline__ uint64_t twice32(uint32_t x) {
    return (uint64_t)twice16(x & 0xFFFFu) | ((uint64_t)twice16(x >> 16) << 32);
}

// v of lane l (l wave-uniform)
__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int l) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32;
}

// The runs of which some block is in s: their blocks above the lowest set one
// (carry of an addition through the connection bits) ...
__device__ __forceinline__ uint64_t fill_up(uint64_t conn, uint64_t s) {
    const uint64_t y = (s << 1) & conn;
    return s | y | (conn & ~(conn + y));
}
// ... and the starts of those runs (the same carry in the mirrored row).
__device__ __forceinline__ uint64_t starts_of(uint64_t conn, uint64_t s) {
    const uint64_t c = __builtin_bitreverse64(conn), r = __builtin_bitreverse64(s);
    return __builtin_bitreverse64(((c + (r & c)) | r) & ~c);
}

// LDS forest of a group: entry v = row * 65 + start column (one extra slot per
// row so that the rows' entries of one column lie in different banks).
constexpr int kRowStep = 65;
__device__ __forceinline__ int forest_row(int v) { return (int)(((uint32_t)v * 4033u) >> 18); }  // v / 65, v < 64 * 65
constexpr int kForest = 64 * 65;

// A lane's CW columns c0 .. c0 + CW - 1 of a row, and one more on each side, as a
// 32-bit window: bit i is column c0 - 1 + i.  The loops over runs and contacts
// work on windows, in half the instructions of 64-bit masks.
template <int CW>
struct Window {
    static_assert(CW <= 16, "a window has 32 bits");
    static constexpr uint32_t kOwn = ((1u << CW) - 1u) << 1;
    int c0;
    __device__ __forceinline__ uint32_t of(uint64_t x) const {
        return (c0 > 0 ? (uint32_t)(x >> (c0 - 1)) : (uint32_t)x << 1) & ((1u << (CW + 2)) - 1u);
    }
    __device__ __forceinline__ uint32_t own(uint64_t x) const { return of(x) & kOwn; }
    __device__ __forceinline__ int col(int i) const { return c0 - 1 + i; }
};
// Start columns of the runs of a row by window bit.
struct RunStarts {
    uint32_t w;
    int in;  // start of a run that reaches the window from the left
    __device__ __forceinline__ int operator()(int first_col, int i) const {
        const uint32_t t = w & ((2u << i) - 1u);
        return t ? first_col + 31 - __builtin_clz(t) : in;
    }
};
template <int CW>
__device__ __forceinline__ RunStarts run_starts(const Window<CW> &win, uint64_t starts) {
    return RunStarts{win.of(starts), run_of(starts, max(win.c0 - 1, 0))};
}

__device__ __forceinline__ uint64_t keep_of(const Geo &g, int word) { return word == g.wpr - 1 ? g.tail : ~0ull; }

// Root of node id: at most `cap` steps; ok is cleared when the cap stops the
// walk (the ancestor reached so far is returned).
__device__ __forceinline__ int node_root(const VLG_GLOBAL int32_t *par, int id, int p, int cap, bool &ok) {
    for (int it = 0; p != id; it++) {
        if (it >= cap) {
            ok = false;
            break;
        }
        id = p;
        p = par[id];
    }
    return id;
}

// The roots of id[0 .. N) by walks in lockstep, so that their loads overlap
// (entries that are done load their root again).
template <int N>
__device__ __forceinline__ void node_roots(const VLG_GLOBAL int32_t *par, int (&id)[N], int cap, bool &ok) {
    int p[N];
#pragma unroll
    for (int j = 0; j < N; j++) p[j] = par[id[j]];
    for (int it = 0;; it++) {
        bool done = true;
#pragma unroll
        for (int j = 0; j < N; j++) done &= p[j] == id[j];
        if (done) break;
        if (it >= cap) {
            ok = false;
            break;
        }
#pragma unroll
        for (int j = 0; j < N; j++) {
            id[j] = p[j];
            p[j] = par[p[j]];
        }
    }
}

// x without its n lowest set bits
template <int N>
__device__ __forceinline__ uint64_t drop_bits(uint64_t x) {
#pragma unroll
    for (int j = 0; j < N; j++) x &= x - 1;
    return x;
}

// Union of a and b on the LDS forest (L[x] <= x, a root is the smallest entry
// of its set).  Both walks advance together, one path-halving step per round,
// so their LDS latencies overlap; once both reach roots the larger root is
// hooked under the smaller with atomicMin, and if that root was hooked
// meanwhile the returned parent is united in its place.  Halving stores may
// race with other lanes' hooks; the hooking lane then unites the old parent
// as well, so no connection is lost.  At most `cap` rounds: returns false
// when the cap stops the walk (the union may be missing).
__device__ __forceinline__ bool lds_unite(int *L, int a, int b, int cap) {
    for (int it = 0; a != b; it++) {
        if (it >= cap) return false;
        const int pa = lds_ld(&L[a]), pb = lds_ld(&L[b]);
        if (pa == a && pb == b) {
            const int hi = a > b ? a : b, lo = a > b ? b : a;
            const int old = atomicMin(&L[hi], lo);
            if (old == hi) return true;
            a = old;
            b = lo;
            continue;
        }
        const int ga = pa != a ? lds_ld(&L[pa]) : pa, gb = pb != b ? lds_ld(&L[pb]) : pb;
        if (pa != a) {
            if (ga != pa) L[a] = ga;
            a = ga;
        }
        if (pb != b) {
            if (gb != pb) L[b] = gb;
            b = gb;
        }
    }
    return true;
}

// ------------------------------------------------------------------ global forest
// Global union-find over the nodes.  A root is hooked under the root of
// smaller priority uf_prio(id), a bijective mix of the id, so the priority
// strictly falls along every parent path.  Linking by id instead turns a row
// of tiles whose components join left to right (a corridor crossing the
// image) into a chain as long as the row, because every tile hooks under its
// left neighbour at the same time; pseudo-random priorities keep the expected
// depth logarithmic.  Node 0 (meets the seeds) has the smallest priority and
// is never hooked.  Plain loads and stores may see stale values (the L2 of
// one XCD is not coherent with another's within a kernel); that costs
// retries, never correctness: every value ever stored in P[x] is an ancestor
// of x, sets only grow, and a hook is a compare-and-swap that succeeds only
// on a current root and otherwise hands back the current parent, which is
// then united in turn.
// MIXED (images): the ids are of nodes, a fixed stride apart in neighbouring
// tiles, and after one multiplication by the golden ratio alone their priorities
// ran monotonically over whole rows of tiles at a stride of 144: lines across
// a 64 x 60000 image were chains of over 192 nodes, 16 with a second round of
// mixing.  Volumes (ids of blocks, tiles 64 apart) keep one round: merging a coin
// mask of 256^3 takes 109 us with it, 170 with two.
template <bool MIXED>
__device__ __forceinline__ uint32_t uf_prio(int x) {
    uint32_t h = (uint32_t)x * 0x9E3779B1u;  // odd multipliers and xor-shifts: bijections, 0 stays 0
    if (MIXED) h = (h ^ (h >> 15)) * 0x85EBCA77u;
    return h ^ (h >> 16);
}

// The roots of a and b, walked in lockstep (path halving on both) so that the
// loads of the two paths overlap.  `budget` counts the rounds left to the
// caller's walk; returns false when it runs out.
__device__ __forceinline__ bool g_find2(VLG_GLOBAL int *P, int &a, int &b, int &budget) {
    while (true) {
        if (--budget < 0) return false;
        const int pa = P[a], pb = P[b];
        if (pa == a && pb == b) return true;
        const int ga = P[pa], gb = P[pb];
        if (pa != a) {
            if (ga != pa) P[a] = ga;
            a = ga;
        }
        if (pb != b) {
            if (gb != pb) P[b] = gb;
            b = gb;
        }
    }
}

// Unite a and b; returns the number of hook attempts, and clears ok when the
// walk used up `cap` rounds (finds and hooks together) before it finished.
template <bool MIXED>
__device__ int g_unite(VLG_GLOBAL int *P, int a, int b, int cap, bool &ok) {
    int tries = 0, budget = cap;
    while (true) {
        tries++;
        if (!g_find2(P, a, b, budget)) {
            ok = false;
            return tries;
        }
        if (a == b) return tries;
        if (uf_prio<MIXED>(a) < uf_prio<MIXED>(b)) {
            const int t = a;
            a = b;
            b = t;
        }
        int old = a;  // hook a (larger priority) under b if a is still a root
        __hip_atomic_compare_exchange_strong(&P[a], &old, b, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        if (old == a) return tries;
        a = old;
    }
}

// Set a seed bit of root id.
__device__ __forceinline__ void flag_or(VLG_GLOBAL uint8_t *flag, int id, uint32_t bit) {
    VLG_GLOBAL uint8_t *p = flag + id;
    const uint32_t k = (uint32_t)(uintptr_t)p & 3u;
    if (!(*p & bit))
        __hip_atomic_fetch_or((VLG_GLOBAL uint32_t *)(p - k), bit << (8 * k), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace
}  // namespace vlg
