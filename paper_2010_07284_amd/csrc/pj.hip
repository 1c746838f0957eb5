// pj.hip -- the paper's own connected-component labelling (Sect. 3, Alg. CCL):
// coordinate labels, max-neighbour pointer jumping (mainIteration), a
// periodic reconnect with an atomic write, and a termination check the host
// waits on; plus the reachability steps (seed flags, gather) on its labels.
//
// Labels are 32-bit keys ((row << 16) | column) + 1, so the key order is the
// lexicographic order of (row, column) pairs, and 0 is null (below every
// pair).  Rows and columns must stay below 65535.  Label arrays are
// row-major [H][W]; background pixels hold 0 in both ping-pong buffers from
// initialization on and are never written again.
//
// A wave has kPjRows words of one mask column, kPjRows rows down: lane l owns
// pixel 64*w + l of each of those rows.  A label array of 2048^2 pixels stays
// in the last-level cache, and a wave of one row is bound by its chain of
// dependent loads; the loads of four rows are in flight together, and rows
// shared by the 3 x 3 neighbourhoods are loaded once, with the neighbouring
// lanes' values for the columns beside: reconnect 27 -> 9.6 us, check 17 -> 7.0, copy
// 10.3 -> 7.0 (2 rows: 11.3, 9.5, 8.9; 8 rows: 9.0, 6.1, 6.0 but half the waves
// for small images).
// A wave whose words have no pixel of the labelled set returns at once.
#include "dev.h"

namespace vlg {
namespace {

constexpr int kPjThreads = 256;
constexpr int kPjWaves = kPjThreads / 64;
constexpr int kPjRows = 4;

// The word of operand r at (row, w), complement applied, padding bits 0;
// 0 outside the image.
__device__ __forceinline__ uint64_t pj_word(const Geo &g, const MRef &r, int row, int w) {
    if (row < 0 || row >= g.H || w < 0 || w >= g.wpr) return 0ull;
    const uint64_t v = (r.p ? glb(r.p)[(int64_t)row * g.wpr + w] : 0ull) ^ r.inv;
    return w == g.wpr - 1 ? (v & g.tail) : v;
}
__device__ __forceinline__ uint64_t pj_lane64(uint64_t v, int l) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32;
}

__device__ __forceinline__ uint32_t pj_key(int row, int col) { return (((uint32_t)row << 16) | (uint32_t)col) + 1u; }
__device__ __forceinline__ int64_t pj_index(const Geo &g, uint32_t key) {
    const uint32_t k = key - 1u;
    return (int64_t)(k >> 16) * g.W + (k & 0xFFFFu);
}

// This wave's rows row0 .. row0 + kPjRows - 1, word w, pixel column and the
// words of the labelled set b.  Returns false (wave-uniform) for waves past
// the row's last word.
struct PjPos {
    int row0, w, col, lane;
    uint64_t bw[kPjRows];
    bool any;  // some word is not 0
    __device__ __forceinline__ bool mine(int i) const { return (bw[i] >> lane) & 1ull; }
    __device__ __forceinline__ int row(const Geo &g, int i) const { return min(max(row0 + i, 0), g.H - 1); }
    __device__ __forceinline__ int64_t at(const Geo &g, int i) const { return (int64_t)(row0 + i) * g.W + col; }
};
__device__ __forceinline__ bool pj_pos(const Geo &g, const MRef &b, PjPos &q) {
    const int nx = (g.wpr + kPjWaves - 1) / kPjWaves, k = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    q.row0 = k / nx * kPjRows;
    q.w = k % nx * kPjWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (q.w >= g.wpr) return false;
    q.lane = (int)(threadIdx.x & 63);
    q.col = q.w * 64 + q.lane;
    const uint64_t v = pj_word(g, b, q.row0 + (q.lane & (kPjRows - 1)), q.w);
    q.any = __any(v != 0);
#pragma unroll
    for (int i = 0; i < kPjRows; i++) q.bw[i] = pj_lane64(v, i);
    return true;
}

// The labels of rows row0 + first .. of this wave's columns (rows and columns
// clamped into the image: a pixel's neighbourhood then holds some pixels
// twice, never one outside it), with those of the columns to the left and
// right.  Called by all lanes.
template <int N>
struct PjLabels {
    uint32_t l[N], c[N], r[N];
};
template <int N>
__device__ __forceinline__ void pj_rows(const Geo &g, const PjPos &q, const uint32_t *__restrict__ lab, int first,
                                        PjLabels<N> &v) {
    const int col = min(q.col, g.W - 1), halo = q.lane < 32 ? max(q.w * 64 - 1, 0) : min(q.w * 64 + 64, g.W - 1);
    uint32_t e[N];
#pragma unroll
    for (int j = 0; j < N; j++) {
        const VLG_GLOBAL uint32_t *p = glb(lab) + (int64_t)q.row(g, first + j) * g.W;
        v.c[j] = p[col];
        e[j] = p[halo];
    }
#pragma unroll
    for (int j = 0; j < N; j++) {
        const uint32_t lp = (uint32_t)lane_prev((int)v.c[j]), ln = (uint32_t)lane_next((int)v.c[j]);
        v.l[j] = q.lane == 0 ? e[j] : lp;
        v.r[j] = q.lane == 63 ? e[j] : ln;
    }
}
__device__ __forceinline__ uint32_t max3(uint32_t a, uint32_t b, uint32_t c) { return max(max(a, b), c); }

// Nothing left to do: the termination check before this round passed.  The
// host enqueues a part of a round before it has seen that check.
__device__ __forceinline__ bool pj_done(const uint32_t *go) { return go && glb(go)[0] == 0u; }

__global__ __launch_bounds__(kPjThreads) void k_pj_init(Geo g, MRef b, uint32_t *a_, uint32_t *b_, uint32_t *term) {
    PjPos q;
    if (blockIdx.x == 0 && threadIdx.x == 0) glb(term)[0] = 0u;
    if (!pj_pos(g, b, q) || q.col >= g.W) return;
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        if (q.row0 + i >= g.H) break;
        const uint32_t key = q.mine(i) ? pj_key(q.row0 + i, q.col) : 0u;
        glb(a_)[q.at(g, i)] = key;
        glb(b_)[q.at(g, i)] = key;
    }
}

// mainIteration: a pixel holding (i', j') takes the largest label around (i', j').
// The targets of a wave's pixels scatter, and every load instruction goes
// line by line: three 12-byte loads (rows of at least 3 pixels, W3) instead of
// nine of 4 bytes, 11.9 us instead of 19.5 (one row per wave: 21.2) at 2048^2,
// where reading and writing the labels once takes 6.6.
template <bool W3>
__global__ __launch_bounds__(kPjThreads) void k_pj_main(Geo g, MRef b, const uint32_t *__restrict__ in,
                                                      uint32_t *__restrict__ out, const uint32_t *go) {
    typedef uint32_t u3 __attribute__((ext_vector_type(3), aligned(4)));
    PjPos q;
    if (pj_done(go) || !pj_pos(g, b, q) || !q.any) return;
    const VLG_GLOBAL uint32_t *lab = glb(in);
    const int colc = min(q.col, g.W - 1);
    uint32_t t[kPjRows], m[kPjRows];
#pragma unroll
    for (int i = 0; i < kPjRows; i++) t[i] = lab[(int64_t)q.row(g, i) * g.W + colc];
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        // background lanes look around themselves, next to their neighbours
        const int tr = q.mine(i) ? (int)((t[i] - 1u) >> 16) : q.row(g, i);
        const int tc = q.mine(i) ? (int)((t[i] - 1u) & 0xFFFFu) : colc;
        const VLG_GLOBAL uint32_t *p = lab + (int64_t)tr * g.W;
        const VLG_GLOBAL uint32_t *u = tr > 0 ? p - g.W : p, *d = tr < g.H - 1 ? p + g.W : p;
        if (W3) {
            // in the first and last column the outer one of the three is no neighbour
            const int c = min(max(tc - 1, 0), g.W - 3);
            const u3 x = *(const VLG_GLOBAL u3 *)(u + c), y = *(const VLG_GLOBAL u3 *)(p + c),
                     z = *(const VLG_GLOBAL u3 *)(d + c);
            const uint32_t l = max3(x[0], y[0], z[0]), o = max3(x[1], y[1], z[1]), r = max3(x[2], y[2], z[2]);
            m[i] = max3(tc == g.W - 1 ? 0u : l, o, tc == 0 ? 0u : r);
        } else {
            const int c0 = max(tc - 1, 0), c2 = min(tc + 1, g.W - 1);
            m[i] = max3(max3(u[c0], u[tc], u[c2]), max3(p[c0], p[tc], p[c2]), max3(d[c0], d[tc], d[c2]));
        }
    }
#pragma unroll
    for (int i = 0; i < kPjRows; i++)
        if (q.mine(i)) glb(out)[q.at(g, i)] = m[i];
}

// reconnect, first half: the output starts as a copy of the input labels.
__global__ __launch_bounds__(kPjThreads) void k_pj_copy(Geo g, MRef b, const uint32_t *__restrict__ in,
                                                      uint32_t *__restrict__ out) {
    PjPos q;
    if (!pj_pos(g, b, q) || !q.any || q.col >= g.W) return;
    uint32_t t[kPjRows];
#pragma unroll
    for (int i = 0; i < kPjRows; i++) t[i] = glb(in)[(int64_t)q.row(g, i) * g.W + q.col];
#pragma unroll
    for (int i = 0; i < kPjRows; i++)
        if (q.mine(i)) glb(out)[q.at(g, i)] = t[i];
}

// reconnect, second half: the largest label around the pixel, when above the
// label stored at the pixel it points to, is written there by atomic
// maximum (several pixels may point to the same one).  Reads only `in`.
__global__ __launch_bounds__(kPjThreads) void k_pj_reconnect(Geo g, MRef b, const uint32_t *__restrict__ in,
                                                           uint32_t *out) {
    PjPos q;
    if (!pj_pos(g, b, q) || !q.any) return;
    PjLabels<kPjRows + 2> v;
    pj_rows(g, q, in, -1, v);
    uint32_t cd[kPjRows];
    int64_t ti[kPjRows];
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        ti[i] = q.mine(i) ? pj_index(g, v.c[i + 1]) : 0;
        cd[i] = glb(in)[ti[i]];
    }
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        const uint32_t ab = max3(max3(v.l[i], v.c[i], v.r[i]), max3(v.l[i + 1], v.c[i + 1], v.r[i + 1]),
                                 max3(v.l[i + 2], v.c[i + 2], v.r[i + 2]));
        if (q.mine(i) && ab > cd[i])
            __hip_atomic_fetch_max(glb(out) + ti[i], ab, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Termination check: does any pixel of b have a neighbour of b with another
// label?  Each pair of neighbours is compared once (right, and the three
// below); a background neighbour holds 0 and is not compared.  (Below the
// last row the row itself is compared, whose pixels are neighbours too.)
__global__ __launch_bounds__(kPjThreads) void k_pj_check(Geo g, MRef b, const uint32_t *__restrict__ lab,
                                                       uint32_t *term) {
    PjPos q;
    if (!pj_pos(g, b, q) || !q.any) return;
    PjLabels<kPjRows + 1> v;
    pj_rows(g, q, lab, 0, v);
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        auto differs = [&](uint32_t u) { return u != 0u && u != v.c[i]; };
        bad |= q.mine(i) && (differs(v.r[i]) || differs(v.l[i + 1]) || differs(v.c[i + 1]) || differs(v.r[i + 1]));
    }
    const uint64_t any = __ballot(bad);
    if (any && q.lane == __builtin_ctzll(any)) glb(term)[0] = 1u;
}

// The check's result to the host's word, and the next round's check word cleared.
__global__ void k_pj_publish(const uint32_t *term, uint32_t *next, uint32_t *host) {
    if (threadIdx.x != 0) return;
    __hip_atomic_store(glb(host), glb(term)[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    glb(next)[0] = 0u;
}

// Seeds of a reachability: flag the labels of the pixels of N(y & z) & b.
__global__ __launch_bounds__(kPjThreads) void k_pj_seed(Geo g, MRef b, MRef y, MRef z,
                                                      const uint32_t *__restrict__ lab, uint8_t *flag,
                                                      uint32_t bit) {
    PjPos q;
    if (!pj_pos(g, b, q) || !q.any) return;
    uint64_t n = 0;  // lane j: the row row0 - 1 + j, widened by one column
    if (q.lane < kPjRows + 2) {
        const int r = q.row0 - 1 + q.lane;
        const uint64_t c = pj_word(g, y, r, q.w) & pj_word(g, z, r, q.w);
        const uint64_t l = pj_word(g, y, r, q.w - 1) & pj_word(g, z, r, q.w - 1);
        const uint64_t h = pj_word(g, y, r, q.w + 1) & pj_word(g, z, r, q.w + 1);
        n = c | (c << 1) | (c >> 1) | (l >> 63) | (h << 63);
    }
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        const uint64_t s = (pj_lane64(n, i) | pj_lane64(n, i + 1) | pj_lane64(n, i + 2)) & q.bw[i];
        if (!((s >> q.lane) & 1ull)) continue;
        VLG_GLOBAL uint8_t *f = glb(flag) + pj_index(g, glb(lab)[q.at(g, i)]);
        if (!(*f & bit)) *f = (uint8_t)(*f | bit);
    }
}

// Another seed set on the same labelling: flag the labels of the pixels of
// the mask s (a subset of the labelled set, N(seeds) & b).
__global__ __launch_bounds__(kPjThreads) void k_pj_reseed(Geo g, MRef s, const uint32_t *__restrict__ lab,
                                                        uint8_t *flag, uint32_t bit) {
    PjPos q;
    if (!pj_pos(g, s, q) || !q.any) return;
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        const uint32_t key = q.mine(i) ? glb(lab)[q.at(g, i)] : 0u;
        if (key == 0u) continue;
        VLG_GLOBAL uint8_t *f = glb(flag) + pj_index(g, key);
        if (!(*f & bit)) *f = (uint8_t)(*f | bit);
    }
}

// out = (y & z) | (pixels of b whose label carries `bit`)
__global__ __launch_bounds__(kPjThreads) void k_pj_gather(Geo g, MRef b, MRef y, MRef z,
                                                        const uint32_t *__restrict__ lab,
                                                        const uint8_t *__restrict__ flag, uint32_t bit,
                                                        uint64_t *out) {
    PjPos q;
    if (!pj_pos(g, b, q)) return;
    uint32_t t[kPjRows];
#pragma unroll
    for (int i = 0; i < kPjRows; i++) t[i] = q.mine(i) ? glb(lab)[q.at(g, i)] : 0u;
    uint64_t zw = 0;  // lane i: the pixels of row i
#pragma unroll
    for (int i = 0; i < kPjRows; i++) {
        const uint64_t v = __ballot(q.mine(i) && (glb(flag)[q.mine(i) ? pj_index(g, t[i]) : 0] & bit) != 0);
        if (q.lane == i) zw = v;
    }
    const int row = q.row0 + q.lane;
    if (q.lane < kPjRows && row < g.H)
        glb(out)[(int64_t)row * g.wpr + q.w] = (pj_word(g, y, row, q.w) & pj_word(g, z, row, q.w)) | zw;
}

// Keys to row-major indices (y*W + x of the label's pixel), -1 for null.
__global__ __launch_bounds__(kPjThreads) void k_pj_labels(Geo g, const uint32_t *__restrict__ lab,
                                                        int32_t *__restrict__ labels) {
    const int64_t i = (int64_t)blockIdx.x * kPjThreads + threadIdx.x, n = (int64_t)g.H * g.W;
    if (i >= n) return;
    const uint32_t key = glb(lab)[i];
    glb(labels)[i] = key == 0u ? -1 : (int32_t)pj_index(g, key);
}

__global__ __launch_bounds__(kPjThreads) void k_pj_fill(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kPjThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kPjThreads)
        glb(p)[i] = v;
}

int pj_blocks(int64_t n, int cap) {
    int64_t b = (n + kPjThreads - 1) / kPjThreads;
    return (int)(b < 1 ? 1 : b > cap ? cap : b);
}

unsigned pj_grid(const Geo &g) {
    return (unsigned)(((g.wpr + kPjWaves - 1) / kPjWaves) * ((g.H + kPjRows - 1) / kPjRows));
}

}  // namespace

bool pj_shape_ok(int H, int W) { return H < 65535 && W < 65535; }

hipError_t launch_pj_init(hipStream_t s, const Geo &g, MRef b, const PjWork &w) {
    if (g.nwords == 0) return hipSuccess;
    k_pj_init<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[0], w.lab[1], w.term);
    return hipGetLastError();
}

hipError_t launch_pj_main(hipStream_t s, const Geo &g, MRef b, const PjWork &w, int from, const uint32_t *go) {
    if (g.nwords == 0) return hipSuccess;
    if (g.W >= 3)
        k_pj_main<true><<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[from], w.lab[1 - from], go);
    else
        k_pj_main<false><<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[from], w.lab[1 - from], go);
    return hipGetLastError();
}

hipError_t launch_pj_reconnect(hipStream_t s, const Geo &g, MRef b, const PjWork &w, int from) {
    if (g.nwords == 0) return hipSuccess;
    k_pj_copy<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[from], w.lab[1 - from]);
    k_pj_reconnect<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[from], w.lab[1 - from]);
    return hipGetLastError();
}

hipError_t launch_pj_check(hipStream_t s, const Geo &g, MRef b, const PjWork &w, int at, int64_t round,
                           uint32_t *host) {
    if (g.nwords == 0) return hipSuccess;
    uint32_t *term = w.term + (round & 1), *next = w.term + (~round & 1);
    k_pj_check<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, w.lab[at], term);
    k_pj_publish<<<1, 64, 0, s>>>(term, next, host);
    return hipGetLastError();
}

hipError_t launch_pj_clear_flags(hipStream_t s, const Geo &g, const PjWork &w) {
    const int64_t n = ((int64_t)g.H * g.W + 3) / 4;
    if (n == 0) return hipSuccess;
    k_pj_fill<<<(unsigned)pj_blocks(n, 8192), kPjThreads, 0, s>>>((uint32_t *)w.flag, n, 0u);
    return hipGetLastError();
}

hipError_t launch_pj_seed(hipStream_t s, const Geo &g, MRef b, MRef y, MRef z, const PjWork &w, int at, int user) {
    if (g.nwords == 0) return hipSuccess;
    k_pj_seed<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, y, z, w.lab[at], w.flag, 2u << user);
    return hipGetLastError();
}

hipError_t launch_pj_reseed(hipStream_t s, const Geo &g, MRef sm, const PjWork &w, int at, int user) {
    if (g.nwords == 0) return hipSuccess;
    k_pj_reseed<<<pj_grid(g), kPjThreads, 0, s>>>(g, sm, w.lab[at], w.flag, 2u << user);
    return hipGetLastError();
}

hipError_t launch_pj_gather(hipStream_t s, const Geo &g, MRef b, MRef y, MRef z, const PjWork &w, int at, int user,
                            uint64_t *out) {
    if (g.nwords == 0) return hipSuccess;
    k_pj_gather<<<pj_grid(g), kPjThreads, 0, s>>>(g, b, y, z, w.lab[at], w.flag, 2u << user, out);
    return hipGetLastError();
}

hipError_t launch_pj_labels(hipStream_t s, const Geo &g, const PjWork &w, int at, int32_t *labels) {
    const int64_t n = (int64_t)g.H * g.W;
    if (n == 0) return hipSuccess;
    k_pj_labels<<<(unsigned)((n + kPjThreads - 1) / kPjThreads), kPjThreads, 0, s>>>(g, w.lab[at], labels);
    return hipGetLastError();
}

}  // namespace vlg
