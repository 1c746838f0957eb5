// ccl.hip -- connected components on packed masks (gfx950, wave64): the
// labelling behind reachability (rho a[b], paper Sect. 3: label the
// 8-components of b, keep those that meet N a) and the canonical labels of
// vlg_ccl_labels.  Not the paper's iterative pointer jumping (Alg. CCL,
// pj.hip) but union-find in a fixed number of launches without a host wait.
//
// Union-find runs over the runs of 2x2 pixel blocks: any two foreground
// pixels of a block are 8-adjacent, horizontally connected blocks of a block
// row form a run, and a run is handled as one bit range of 64-bit masks.
//
//   local   components of each tile (TBH block rows x 64 blocks) in LDS
//   merge   components that meet across tile borders, in global memory
//   gather  every run asks for its component's seed bit
//
// Tile passes give a lane one block row of one tile, with the 64 blocks of
// the row in 64-bit masks, so mask logic costs one instruction for 64 rows
// of 64 blocks.  A workgroup takes 64 such rows (64 / TBH tiles side by
// side, so the mask rows it reads are whole sectors); its waves hold the same
// rows and share the work by columns or by run number.  A lane per block, as
// before, was bound by VALU issue (some 250 instructions per 64 blocks) and by
// the 5 bytes it wrote per block.  One labelling and gather at 4096^2
// (smoothed noise, 16 block rows per tile): 63 us before (local 21, merge 22,
// flags 9, gather 10), 31 us now (16.5, 8.4, -, 6); at 1024^2: 37 -> 22 us.
//
// Only the components that touch a border shared with another tile (nodes)
// live in global memory: their parents, and the labels of the border blocks,
// in compact per-tile tables.  A run's 16-bit label is its node's rank in the
// tile (bit 15 set), or for inner components the root block (row * 64 +
// column) with bit 14 = it meets the seeds of the labelling's first user.
#include "runs.h"

namespace vlg {
namespace {

constexpr uint32_t kLabNode = 0x8000u, kLabSeed = 0x4000u;

// A group of NR block rows: NR / TBH tiles side by side, 2*TBH pixel rows of SW
// words, NW words in all.  A wave has 64 / NR lanes per row (segments).
template <int TBH, int NR>
struct Grp {
    static constexpr int SUB = NR / TBH;      // tiles side by side
    static constexpr int SEG = 64 / NR;
    static constexpr int SW = 2 * SUB;        // words per pixel row
    static constexpr int PR = 2 * TBH;        // pixel rows
    static constexpr int SBP = SW + 1;        // LDS row strides in words (odd: no bank conflicts
    static constexpr int SAP = SW + 3;        // between the rows of one column)
    static constexpr int NA = (PR + 2) * (SW + 2);  // with a halo of one row and one word
    static constexpr int NW = PR * SW;
    static_assert(NW == 4 * NR && NR >= TBH && NW <= kThreads, "at most one word per thread");
};

// A block row: its blocks' four pixels, and its runs.
struct Row {
    uint64_t t0, t1, b0, b1;  // top-left, top-right, bottom-left, bottom-right pixel of block l
    uint64_t conn;            // block l is connected to block l-1
    uint64_t starts;          // block l starts a run
    __device__ __forceinline__ uint64_t fg() const { return t0 | t1 | b0 | b1; }
};
__device__ __forceinline__ Row make_row(uint64_t t0, uint64_t t1, uint64_t b0, uint64_t b1) {
    Row r{t0, t1, b0, b1, 0, 0};
    r.conn = (t0 | b0) & ((t1 | b1) << 1);
    r.starts = r.fg() & ~r.conn;
    return r;
}
// The masks of the group's rows, written by four waves (wave k: pixel row k>>1
// of the block rows, word k&1 of the tiles), read by all.
struct RowMasks {
    uint32_t e[4][64], o[4][64];
    __device__ __forceinline__ Row row(int lane) const {
        auto two = [&](const uint32_t (&m)[4][64], int k) {
            return (uint64_t)m[k][lane] | ((uint64_t)m[k + 1][lane] << 32);
        };
        return make_row(two(e, 0), two(o, 0), two(e, 2), two(o, 2));
    }
};

// ------------------------------------------------------------------ local
// The components of a group of tiles.  Contacts between runs of consecutive
// rows come out of the masks (a contact is dropped when another contact of
// the same two runs, at the left neighbour or in the same block, remains); a
// run's first contact becomes its parent without a union, the others are
// united from a queue.  Then every run finds its root, roots collect whether
// they touch a shared border and whether they meet the seeds (bit sets per
// row in LDS), and the runs' labels, the nodes and the border tables are
// written.  NW waves, 64 / (NW * SEG) columns of a row per lane.  Bound by chains
// of LDS round trips (of 20 k cycles at 1024^2 smoothed noise: staging 3 k,
// unions 4 k, roots 4 k, border tables 2 k), on large images by VALU issue.
// CANON (vlg_ccl_labels): also the smallest pixel of every component, at its
// node (ncanon) or its root block (icanon).
template <int TBH, int NR, int NW, bool CANON>
__device__ __forceinline__ void ccl_local_group(const Geo &g, const CclGeo &q, const CclArrays &a, const MRef &b,
                                                const MRef &y, const MRef &z, bool multi, int gx, int ty,
                                                const LoopGuard &gd, int32_t *ncanon_, int32_t *icanon_) {
    using G = Grp<TBH, NR>;
    constexpr int NT = 64 * NW, CW = 64 / (NW * G::SEG);  // threads; columns per lane
    constexpr int NAI = (G::NA + NT - 1) / NT;
    // the staged words are dead once the row masks are written, and later tables
    // take their place (26 KB at TBH 32: six groups of four waves per compute
    // unit instead of five, a batch 121.5 -> 113.6 us; seven at 23 KB and one
    // barrier more: 114.4)
    __shared__ union {
        uint64_t b[G::PR * G::SBP];
        struct {
            uint32_t bits[2][64][2];  // roots that touch a shared border; roots that meet the seeds
            uint32_t pre[64];
        };
    } ub;
    __shared__ union {
        uint64_t a[(G::PR + 2) * G::SAP];
        int pairs[NW][128];  // union pairs: entry | entry of the row above << 16
    } ua;
    auto &sb = ub.b;
    auto &sa = ua.a;
    auto &sbits = ub.bits;
    auto &spre = ub.pre;
    auto &pairs = ua.pairs;
    __shared__ RowMasks rm;
    __shared__ uint32_t sseed[4][64];       // blocks with a seed pixel, by pixel row and word as rm
    __shared__ int L[kForest];
    __shared__ int smin[CANON ? kForest : 1];
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));  // per-tile addressing is recomputed, not kept across a persistent loop
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = ty * G::PR, wc0 = gx * G::SW;
    const bool seeds = (y.p || y.inv) && (z.p || z.inv);
    {
        const int p = tid / G::SW, w = tid % G::SW, row = r0 + p, word = wc0 + w;
        // all loads first, from clamped addresses, so that none waits for another
        const bool in = tid < G::NW && row < g.H && word < g.wpr;
        uint64_t v = b.p ? glb(b.p)[in ? (int64_t)row * g.wpr + word : 0] : 0ull;
        uint64_t s[NAI], t[NAI];
        bool sin[NAI];
        if (seeds) {
#pragma unroll
            for (int k = 0; k < NAI; k++) {
                const int i = tid + k * NT, yy = r0 + i / (G::SW + 2) - 1, ww = wc0 + i % (G::SW + 2) - 1;
                sin[k] = i < G::NA && yy >= 0 && yy < g.H && ww >= 0 && ww < g.wpr;
                const int64_t x = sin[k] ? (int64_t)yy * g.wpr + ww : 0;
                s[k] = y.p ? glb(y.p)[x] : 0ull;
                t[k] = z.p ? glb(z.p)[x] : 0ull;
            }
        }
#pragma unroll
        for (int k = 0; k < (NR * kRowStep + NT - 1) / NT; k++) {
            const int x = tid + k * NT;
            if (x >= NR * kRowStep) break;
            L[x] = x;
            if (CANON) smin[x] = 0x7fffffff;
        }
        if (tid < G::NW) sb[p * G::SBP + w] = in ? (v ^ b.inv) & keep_of(g, word) : 0ull;
        if (seeds) {
#pragma unroll
            for (int k = 0; k < NAI; k++) {
                const int i = tid + k * NT;
                const int ww = wc0 + i % (G::SW + 2) - 1;
                if (i < G::NA)
                    sa[i / (G::SW + 2) * G::SAP + i % (G::SW + 2)] =
                        sin[k] ? (s[k] ^ y.inv) & (t[k] ^ z.inv) & keep_of(g, ww) : 0ull;
            }
        }
    }
    __syncthreads();
    // this lane's row and its segment of the columns
    const int lr = lane % NR, seg = lane / NR, sub = lr / TBH, rr = lr % TBH;
    if (tid < G::NW) {
        const int k = tid / NR, p = 2 * rr + (k >> 1), w = 2 * sub + (k & 1);
        const uint64_t bw = sb[p * G::SBP + w];
        uint32_t e, o;
        split_even_odd(bw, e, o);
        rm.e[k][lr] = e;
        rm.o[k][lr] = o;
        if (seeds) {
            uint64_t l = 0, c = 0, r = 0;
#pragma unroll
            for (int d = 0; d < 3; d++) {
                const uint64_t *s = &sa[(p + d) * G::SAP + w];
                l |= s[0];
                c |= s[1];
                r |= s[2];
            }
            const uint64_t n = (c | (c << 1) | (c >> 1) | (l >> 63) | (r << 63)) & bw;
            sseed[k][lr] = even_bits(n | (n >> 1));
        }
    }
    __syncthreads();

    if (tid < 256) (&sbits[0][0][0])[tid] = 0;
    // the row (the same in every wave) and the row above it
    const Row m = rm.row(lr);
    const int tx = gx * G::SUB + sub, by = ty * TBH + rr, tile = ty * q.ntx + tx;
    const int c0 = CW * (wave * G::SEG + seg);  // this lane's columns
    const Window<CW> win{c0};
    const int row0 = lr * kRowStep;
    const RunStarts sm = run_starts(win, m.starts);
    bool ok = true;
    {
        // (lane shifts outside any branch: every lane has to take part)
        const uint64_t p0 = lane_prev64(m.b0), p1 = lane_prev64(m.b1), uc = lane_prev64(m.conn),
                       us = lane_prev64(m.starts);
        const uint64_t ub0 = rr ? p0 : 0ull, ub1 = rr ? p1 : 0ull;
        const uint64_t u = (m.t0 | m.t1) & (ub0 | ub1), ul = m.t0 & (ub1 << 1), ur = m.t1 & (ub0 >> 1);
        const uint64_t um64 = u & ~(m.conn & ((uc & (u << 1)) | (ur << 1)));
        const uint64_t lm64 = ul & ~((u & uc) | (m.conn & (u << 1)));
        const uint64_t rm64 = ur & ~(u & (uc >> 1));
        // A run's first contact makes the touched run its parent at once (no
        // one else writes its entry before the barrier); only the others are
        // unions.
        const uint64_t all = um64 | lm64 | rm64;
        const uint32_t f = win.own(all & ~(m.conn & (fill_up(m.conn, all) << 1)));
        const RunStarts su = run_starts(win, us);
        // this row's run at window bit i, the upper row's at bit i
        auto here = [&](int i) { return row0 + sm(c0 - 1, i); };
        auto above = [&](int i) { return row0 - kRowStep + su(c0 - 1, i); };
        uint32_t um = win.own(um64), lm = win.own(lm64), rm_ = win.own(rm64);
        for (uint32_t x = f; x; x &= x - 1) {
            const int i = __builtin_ctz(x);
            L[here(i)] = above(i + ((um >> i) & 1 ? 0 : (lm >> i) & 1 ? -1 : 1));
        }
        rm_ &= ~(f & ~(um | lm));
        lm &= ~(f & ~um);
        um &= ~f;
        __syncthreads();
        // The pairs go through a queue, so that a row with many of them does
        // not hold up the wave: every round appends at most one pair per
        // lane, and whenever 64 are there each lane unites one.
        int n = 0;  // wave-uniform
        auto take = [&](int cnt) {
            wave_lds_handoff();
            n -= cnt;
            if (lane < cnt) {
                const int pr = pairs[wave][n + lane];
                ok &= lds_unite(L, pr & 0xFFFF, pr >> 16, gd.cap);
            }
            wave_lds_handoff();
        };
        for (;;) {
            const uint32_t x = um | lm | rm_;
            const uint64_t act = __ballot(x != 0);
            if (!act) break;
            if (x) {
                const int i = __builtin_ctz(x);
                const uint32_t bit = x & (0u - x), isu = um & bit, isl = isu | (lm & bit);
                const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0u));
                pairs[wave][at] = here(i) | above(i + (isu ? 0 : isl ? -1 : 1)) << 16;
                um &= ~bit;
                if (!isu) lm &= ~bit;
                if (!isl) rm_ &= ~bit;
            }
            n += __popcll(act);
            if (n >= 64) take(64);
        }
        if (n > 0) take(n);
    }
    __syncthreads();

    // every run's root
    uint64_t bs = 0, ss = 0;
    if ((rr == 0 && ty > 0) || (rr == TBH - 1 && ty < q.nty - 1)) bs = m.starts;
    if (tx > 0) bs |= m.starts & 1ull;
    if (tx < q.ntx - 1 && (m.fg() >> 63)) bs |= 1ull << run_of(m.starts, 63);
    if (seeds) {
        const uint64_t s = (uint64_t)(sseed[0][lr] | sseed[2][lr]) |
                           ((uint64_t)(sseed[1][lr] | sseed[3][lr]) << 32);
        ss = starts_of(m.conn, s);
    }
    // Two runs at a time, so that their walks overlap; path halving through
    // atomicMin: a stale store never replaces a root that a run's own lane
    // has written.
    const uint32_t bsw = win.of(bs), ssw = win.of(ss);
    for (uint32_t st = sm.w & win.kOwn; st;) {
        int s[2], x[2];
        s[0] = __builtin_ctz(st);
        st &= st - 1;
        const int nr = st ? 2 : 1;
        s[1] = st ? __builtin_ctz(st) : s[0];
        st &= st - 1;
        x[0] = row0 + win.col(s[0]);
        x[1] = row0 + win.col(s[1]);
        for (int it = 0;; it++) {
            const int p0 = lds_ld(&L[x[0]]), p1 = lds_ld(&L[x[1]]);
            if (p0 == x[0] && p1 == x[1]) break;
            if (it >= gd.cap) {
                ok = false;
                break;
            }
            const int g0 = lds_ld(&L[p0]), g1 = lds_ld(&L[p1]);
            if (g0 != p0) atomicMin(&L[x[0]], g0);
            if (g1 != p1) atomicMin(&L[x[1]], g1);
            x[0] = g0;
            x[1] = g1;
        }
#pragma unroll
        for (int j = 0; j < 2; j++) {
            if (j >= nr) break;
            const int v = row0 + win.col(s[j]), xr = forest_row(x[j]), xc = x[j] - xr * kRowStep;
            if (x[j] != v) L[v] = x[j];
            if ((bsw >> s[j]) & 1) atomicOr(&sbits[0][xr][xc >> 5], 1u << (xc & 31));
            if ((ssw >> s[j]) & 1) atomicOr(&sbits[1][xr][xc >> 5], 1u << (xc & 31));
            if (CANON && xr == lr) {
                // the run's first pixel: in its top pixel row if it has one there
                const uint64_t run = fill_up(m.conn, 1ull << win.col(s[j])), top = (m.t0 | m.t1) & run;
                const int l = __builtin_ctzll(top ? top : (m.b0 | m.b1) & run);
                const int col = 2 * l + ((((top ? m.t0 : m.b0) >> l) & 1) ? 0 : 1);
                atomicMin(&smin[x[j]], (top ? 0 : 128) + col);
            }
        }
    }
    __syncthreads();

    // ranks of the nodes: prefix sums over the rows of each tile
    const uint64_t nodes = (uint64_t)sbits[0][lr][0] | ((uint64_t)sbits[0][lr][1] << 32);
    {
        const int cnt = __popcll(nodes);
        int sum = cnt;
#pragma unroll
        for (int d = 1; d < TBH; d <<= 1) {
            const int t = __shfl_up(sum, d);
            if (rr >= d) sum += t;
        }
        spre[lr] = (uint32_t)(sum - cnt);  // (all waves write the same values)
        if (wave == 0 && seg == 0 && rr == TBH - 1 && tx < q.ntx) glb(a.cnt)[tile] = (uint32_t)sum;
    }
    wave_lds_handoff();
    VLG_GLOBAL uint16_t *lab = glb(a.lab) + (int64_t)by * g.BW + tx * 64;
    const int node0 = tile * q.np + 1;
    int k = __popcll(m.starts & below(c0));
    for (uint32_t st = sm.w & win.kOwn; st; st &= st - 1, k++) {
        const int s = win.col(__builtin_ctz(st)), v = row0 + s;
        const int x = L[v], xr = forest_row(x), xc = x - xr * kRowStep;
        const uint64_t xn = (uint64_t)sbits[0][xr][0] | ((uint64_t)sbits[0][xr][1] << 32);
        uint32_t lb;
        if ((xn >> xc) & 1)
            lb = kLabNode | (spre[xr] + (uint32_t)__popcll(xn & below(xc)));
        else
            lb = (uint32_t)((xr % TBH) * 64 + xc) | (((sbits[1][xr][xc >> 5] >> (xc & 31)) & 1) ? kLabSeed : 0u);
        lab[k] = (uint16_t)lb;
        // (a run whose bit is set is a root unless a walk gave up; its node is
        // set up in either case, so that every label names a valid node)
        if ((nodes >> s) & 1) {
            const int id = node0 + (int)spre[lr] + __popcll(nodes & below(s));
            const bool seeded = (sbits[1][lr][s >> 5] >> (s & 31)) & 1;
            glb(a.par)[id] = seeded && !multi ? 0 : id;
            if (multi) glb(a.flag)[id] = seeded ? 2 : 0;
        }
        if (CANON && x == v) {
            const int px = smin[v];
            const int64_t first = (int64_t)(2 * by + (px >> 7)) * g.W + tx * 128 + (px & 127);
            if ((nodes >> s) & 1)
                glb(ncanon_)[node0 + (int)spre[lr] + __popcll(nodes & below(s))] = (int32_t)first;
            else
                glb(icanon_)[(int64_t)by * g.BW + tx * 64 + s] = (int32_t)first;
        }
        L[v] = (int)lb;
    }
    if (gx == 0 && ty == 0 && tid == 0) glb(a.par)[0] = 0;
    if (q.np > 0) {
        __syncthreads();
        // border tables: rank | block bits << 8, 0 for a background block
        VLG_GLOBAL uint16_t *per = glb(a.per);
        const int side0 = q.ud ? 2 * q.tw : 0;
        if (wave < 2 && seg == 0 && q.lr && tx < q.ntx && rr < q.th) {
            const int l = wave ? 63 : 0;
            uint32_t e = 0;
            if ((m.fg() >> l) & 1) {
                const uint32_t bits = (uint32_t)((m.t0 >> l) & 1) | (uint32_t)((m.t1 >> l) & 1) << 1 |
                                      (uint32_t)((m.b0 >> l) & 1) << 2 | (uint32_t)((m.b1 >> l) & 1) << 3;
                e = (uint32_t)(L[row0 + run_of(m.starts, l)] & 0xFF) | bits << 8;
            }
            per[(int64_t)tile * q.np + side0 + wave * q.th + rr] = (uint16_t)e;
        }
        if (q.ud) {
            const int h = lane >> 5, l = lane & 31;
#pragma unroll
            for (int i = 0; i < (2 * G::SUB + NW - 1) / NW; i++) {
                const int j = min(wave + i * NW, 2 * G::SUB - 1), bottom = j & 1;
                const int jx = gx * G::SUB + (j >> 1), R = (j >> 1) * TBH + (bottom ? TBH - 1 : 0);
                const uint32_t bits = ((rm.e[h][R] >> l) & 1) | ((rm.o[h][R] >> l) & 1) << 1 |
                                      ((rm.e[2 + h][R] >> l) & 1) << 2 | ((rm.o[2 + h][R] >> l) & 1) << 3;
                const int lb = L[R * kRowStep + run_of(read_lane64(m.starts, R), lane)];
                if (lane < q.tw && jx < q.ntx && (bottom ? ty < q.nty - 1 : ty > 0))
                    per[(int64_t)(ty * q.ntx + jx) * q.np + bottom * q.tw + lane] =
                        (uint16_t)(bits ? (uint32_t)(lb & 0xFF) | bits << 8 : 0u);
            }
        }
    }
    guard_report(gd, ok);
}

// ------------------------------------------------------------------ merge
// Two waves per tile: part 0 the top row against the tiles above, part 1 the
// left column against the tile to the left and the right column's upper-right
// contacts against the tile to the right.  Everything a lane needs (labels
// and block bits on both sides of the border) comes from the border tables in
// one round of loads; neighbours along the border from the adjacent lanes.
// The pairs are listed in LDS first and then taken one per lane, so the
// unions of a lane do not follow one another.  A contact between the same two
// nodes as one of the previous lane's is dropped.
constexpr int kMergePairs = 192;  // three contacts per lane
__device__ __forceinline__ void ccl_merge_tile(const Geo &g, const CclGeo &q, const CclArrays &a, int tile, int part,
                                               int2 *pairs, int &unions, int &tries, const LoopGuard &gd) {
    const VLG_GLOBAL uint16_t *per = glb(a.per);
    const int lane = lane_id();
    const int ty = tile / q.ntx, tx = tile - ty * q.ntx;
    const int left0 = q.ud ? 2 * q.tw : 0, right0 = left0 + q.th;
    int my = 0, c[3] = {0, 0, 0};
    auto id = [&](int t, uint32_t e) { return t * q.np + 1 + (int)(e & 0xFF); };
    if (part == 0) {
        if (ty > 0) {
            const int up = tile - q.ntx;
            uint32_t e = 0, u = 0, corner = 0;
            if (lane < q.tw) {
                e = per[(int64_t)tile * q.np + lane];
                u = per[(int64_t)up * q.np + q.tw + lane];
            }
            if (lane == 0 && tx > 0) corner = per[(int64_t)(up - 1) * q.np + q.tw + 63];
            if (lane == 63 && tx < q.ntx - 1) corner = per[(int64_t)(up + 1) * q.np + q.tw];
            uint32_t ul = (uint32_t)lane_prev((int)u), ur = (uint32_t)lane_next((int)u);
            if (lane == 0) ul = corner;
            if (lane == 63) ur = corner;
            const uint32_t bb = e >> 8;
            if (bb) my = id(tile, e);
            if ((bb & 1) && (ul >> 8 & 8)) c[0] = id(lane == 0 ? up - 1 : up, ul);
            if ((bb & 3) && (u >> 8 & 12)) c[1] = id(up, u);
            if ((bb & 2) && (ur >> 8 & 4)) c[2] = id(lane == 63 ? up + 1 : up, ur);
        }
    } else if (q.lr) {
        const int r = lane & 31, right = lane >> 5;
        uint32_t e = 0, n = 0;
        if (r < q.th && (right ? tx < q.ntx - 1 : tx > 0)) {
            e = per[(int64_t)tile * q.np + (right ? right0 : left0) + r];
            n = per[(int64_t)(right ? tile + 1 : tile - 1) * q.np + (right ? left0 : right0) + r];
        }
        const uint32_t pe = (uint32_t)lane_prev((int)e), pn = (uint32_t)lane_prev((int)n);
        const uint32_t bb = e >> 8;
        if (bb) my = id(tile, e);
        if (!right) {
            if ((bb & 5) && (n >> 8 & 10)) c[0] = id(tile - 1, n);
            if (r > 0 && (bb & 1) && (pn >> 8 & 8)) c[1] = id(tile - 1, pn);
        } else if (r > 0 && (bb & 2) && (pn >> 8 & 4)) {
            // redundant when the block above is of this component and touches
            // that same block to its right (a left contact of the right tile)
            const bool covered = (pe & 0xFF) == (e & 0xFF) && (pe >> 8 & 10) && (pn >> 8 & 5);
            if (!covered) c[1] = id(tile + 1, pn);
        }
    }
    const int pm = lane_prev(my), p0 = lane_prev(c[0]), p1 = lane_prev(c[1]), p2 = lane_prev(c[2]);
    if (c[1] == c[0]) c[1] = 0;
    if (c[2] == c[0] || c[2] == c[1]) c[2] = 0;
    int n = 0;  // wave-uniform
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const bool has = c[j] && !(pm == my && (c[j] == p0 || c[j] == p1 || c[j] == p2));
        const uint64_t mask = __ballot(has);
        if (has) {
            const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            pairs[at] = make_int2(my, c[j]);
        }
        n += __popcll(mask);
    }
    wave_lds_handoff();
    bool ok = true;
    for (int i = lane; i < n; i += 64) {
        const int2 pr = pairs[i];
        unions++;
        tries += g_unite<true>(glb(a.par), pr.x, pr.y, gd.cap, ok);
    }
    guard_report(gd, ok);
    wave_lds_handoff();  // the list is rewritten by the wave's next tile
}

// ------------------------------------------------------------------ flags
// Set a seed bit of the lane's root; the active lanes with the first one's root
// (a large component's) once together.
__device__ __forceinline__ void flag_or_wave(VLG_GLOBAL uint8_t *flag, int root, uint32_t bit) {
    const int r0 = __builtin_amdgcn_readfirstlane(root);
    const uint64_t same = __ballot(root == r0);
    if (root != r0 || lane_id() == __builtin_ctzll(same)) flag_or(flag, root, bit);
}

// Carry the first user's seed flags of a tile's nodes to their roots (one
// wave per tile), and point every node at its root: each user's reseed and
// gather walk from there.  (Other waves may meet either parent on their way,
// both lead to the root.)
__device__ __forceinline__ void ccl_flag_tile(const CclGeo &q, const CclArrays &a, int tile, const LoopGuard &gd) {
    VLG_GLOBAL int32_t *par = glb(a.par);
    const int n = (int)glb(a.cnt)[tile], id0 = tile * q.np + 1;
    bool ok = true;
    for (int k = lane_id(); k < n; k += 64) {
        const uint32_t flag = glb(a.flag)[id0 + k];
        const int p = par[id0 + k], root = node_root(par, id0 + k, p, gd.cap, ok);
        if (root != p) par[id0 + k] = root;
        if ((flag & 2) && root != id0 + k) flag_or_wave(glb(a.flag), root, 2u);
    }
    guard_report(gd, ok);
}

// Stage the group's words of x (one per thread, returned; out-of-image bits
// 0) and split them into row masks.  One barrier, before the row masks are
// written: the caller needs another before it reads them.
template <int TBH>
__device__ __forceinline__ uint64_t stage_rows(const Geo &g, const MRef &x, int gx, int ty, int tid, uint64_t *sb,
                                               RowMasks &rm) {
    using G = Grp<TBH, 64>;
    const int p = tid / G::SW, w = tid % G::SW, row = ty * G::PR + p, word = gx * G::SW + w;
    uint64_t v = 0;
    if (row < g.H && word < g.wpr) v = ldm(x, (int64_t)row * g.wpr + word) & keep_of(g, word);
    sb[p * G::SBP + w] = v;
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, sub = lane / TBH, rr = lane % TBH;
    uint32_t e, o;
    split_even_odd(sb[(2 * rr + (wave >> 1)) * G::SBP + 2 * sub + (wave & 1)], e, o);
    rm.e[wave][lane] = e;
    rm.o[wave][lane] = o;
    return v;
}

// Mark, for user u >= 1 of a labelling, the components that meet the seed
// mask y (= N(seeds) & b): inner ones in the tile's useed bits, nodes at their
// roots' flag bytes.
template <int TBH>
__device__ __forceinline__ void ccl_reseed_group(const Geo &g, const CclGeo &q, const CclArrays &a, const MRef &b,
                                                 const MRef &sm, int user, int gx, int ty, const LoopGuard &gd) {
    using G = Grp<TBH, 64>;
    __shared__ uint64_t sb[G::PR * G::SBP];
    __shared__ RowMasks rm, rs;
    __shared__ uint32_t sin[64][2];        // seeded inner roots, by row
    __shared__ uint32_t snode[G::SUB][6];  // seeded nodes, by rank
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 128) (&sin[0][0])[tid] = 0;
    if (tid < G::SUB * 6) (&snode[0][0])[tid] = 0;
    stage_rows<TBH>(g, b, gx, ty, tid, sb, rm);
    __syncthreads();
    stage_rows<TBH>(g, sm, gx, ty, tid, sb, rs);
    __syncthreads();
    const int sub = lane / TBH, rr = lane % TBH, tx = gx * G::SUB + sub, by = ty * TBH + rr;
    const Row m = rm.row(lane);
    const uint64_t ss = starts_of(m.conn, rs.row(lane).fg());
    const VLG_GLOBAL uint16_t *lab = glb(a.lab) + (int64_t)by * g.BW + tx * 64;
    // every fourth seeded run of a row, the labels of four at a time
    uint64_t st = ss;
    for (int i = 0; i < wave; i++) st &= st - 1;
    while (st) {
        uint32_t lb[4];
        int n = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (st) {
                lb[j] = lab[__popcll(m.starts & below(__builtin_ctzll(st)))];
                n++;
            }
            st = drop_bits<4>(st);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (j >= n) break;
            const uint32_t x = lb[j] & 0x7FF;
            uint32_t *at = lb[j] & kLabNode ? &snode[sub][(lb[j] & 0xFF) >> 5]
                                            : &sin[sub * TBH + (int)(x >> 6)][(x >> 5) & 1];
            atomicOr(at, 1u << (lb[j] & 31));
        }
    }
    __syncthreads();
    // useed rows
    if (wave == 0 && tx < q.ntx && by < g.BH) {
        VLG_GLOBAL uint8_t *u = glb(a.useed) + ((int64_t)(ty * q.ntx + tx) * q.th + rr) * q.sb;
        if (q.sb == 8) {
            *(VLG_GLOBAL uint64_t *)u = (uint64_t)sin[lane][0] | ((uint64_t)sin[lane][1] << 32);
        } else {
            for (int j = 0; j < q.sb; j++) u[j] = (uint8_t)(sin[lane][j >> 2] >> (8 * (j & 3)));
        }
    }
    // nodes: 256 / SUB threads per tile
    constexpr int TPS = kThreads / G::SUB;
    const int ns = tid / TPS, nx = gx * G::SUB + ns;
    bool ok = true;
    if (nx < q.ntx) {
        const VLG_GLOBAL int32_t *par = glb(a.par);
        const int t = ty * q.ntx + nx, n = (int)glb(a.cnt)[t], id0 = t * q.np + 1;
        for (int j = tid % TPS; j < n; j += TPS)
            if ((snode[ns][j >> 5] >> (j & 31)) & 1)
                flag_or_wave(glb(a.flag), node_root(par, id0 + j, par[id0 + j], gd.cap, ok), 2u << user);
    }
    guard_report(gd, ok);
}

// ------------------------------------------------------------------ gather
// out = (y & z) | Z, Z = the b-pixels whose component meets the seeds.  The
// nodes' roots are walked once per tile (256 / SUB threads each) into a bit
// table in LDS while the masks are staged; each wave takes every fourth run
// of a row, and a selected run's blocks come out of one carry.  Bound by the
// latency of the walk and of the label loads (the first two labels a wave
// can need are loaded before the masks are known).
template <int TBH>
__device__ __forceinline__ void ccl_gather_group(const Geo &g, const CclGeo &q, const CclArrays &a, const MRef &b,
                                                 const MRef &y, const MRef &z, int user, bool multi, uint64_t *out,
                                                 int gx, int ty, const LoopGuard &gd) {
    using G = Grp<TBH, 64>;
    __shared__ uint64_t sb[G::PR * G::SBP];
    __shared__ RowMasks rm;
    __shared__ uint32_t sin[64][2], sz[64][2];
    __shared__ uint32_t snode[G::SUB][6];
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = lane / TBH, rr = lane % TBH, tx = gx * G::SUB + sub, by = ty * TBH + rr;
    // this thread's output word
    const int p = tid / G::SW, w = tid % G::SW, row = ty * G::PR + p, word = gx * G::SW + w;
    const bool oin = row < g.H && word < g.wpr;
    const int64_t oi = oin ? (int64_t)row * g.wpr + word : 0;
    uint64_t yz = 0;
    if (oin) yz = ldm(y, oi) & ldm(z, oi) & keep_of(g, word);
    // labels of runs wave, wave + 4 of this lane's row
    const int nblk = tx < q.ntx && by < g.BH ? min(64, g.BW - tx * 64) : 0;
    const VLG_GLOBAL uint16_t *lab = glb(a.lab) + (nblk ? (int64_t)by * g.BW + tx * 64 : 0);
    const uint32_t lab0 = wave < nblk ? lab[wave] : 0u, lab1 = wave + 4 < nblk ? lab[wave + 4] : 0u;
    constexpr int TPS = kThreads / G::SUB;
    const int ns = tid / TPS, nk = tid % TPS, nx = gx * G::SUB + ns;
    const VLG_GLOBAL int32_t *par = glb(a.par);
    const int nt = nx < q.ntx ? ty * q.ntx + nx : 0, id0 = nt * q.np + 1;
    const int nn = nx < q.ntx ? (int)glb(a.cnt)[nt] : 0;
    const int first = nk < q.np ? par[id0 + nk] : 0;
    if (tid < 128) {
        (&sz[0][0])[tid] = 0;
        // (th * sb bytes per tile; rows of lanes outside the image are unused)
        uint32_t v = 0;
        if (user > 0) {
            const int R = tid >> 1, rx = gx * G::SUB + R / TBH;
            if (rx < q.ntx && ty * TBH + R % TBH < g.BH) {
                const VLG_GLOBAL uint8_t *u =
                    glb(a.useed) + ((int64_t)(ty * q.ntx + rx) * q.th + R % TBH) * q.sb;
                for (int j = 0; j < 4; j++) {
                    const int at = (tid & 1) * 4 + j;
                    if (at < q.sb) v |= (uint32_t)u[at] << (8 * j);
                }
            }
        }
        (&sin[0][0])[tid] = v;
    }
    if (tid < G::SUB * 6) (&snode[0][0])[tid] = 0;
    const uint64_t bw = stage_rows<TBH>(g, b, gx, ty, tid, sb, rm);  // (its barrier covers the tables above)
    bool ok = true;
    for (int j = nk; j < nn; j += TPS) {
        const int root = node_root(par, id0 + j, j == nk ? first : par[id0 + j], gd.cap, ok);
        if (multi ? (glb(a.flag)[root] >> (1 + user)) & 1 : root == 0) atomicOr(&snode[ns][j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    const Row m = rm.row(lane);
    uint64_t zs = 0, st = m.starts;  // st: the wave's next run is the lowest
    for (int i = 0; i < wave; i++) st &= st - 1;
    auto take = [&](uint32_t lb) {
        if (!st) return;
        const uint32_t x = lb & 0x7FF;
        bool hit;
        if (lb & kLabNode) hit = (snode[sub][(lb & 0xFF) >> 5] >> (lb & 31)) & 1;
        else if (user == 0) hit = lb & kLabSeed;
        else hit = (sin[sub * TBH + (int)(x >> 6)][(x >> 5) & 1] >> (lb & 31)) & 1;
        if (hit) zs |= st & (0 - st);
        st = drop_bits<4>(st);
    };
    take(lab0);
    take(lab1);
    for (int k = wave + 8; st; k += 16) {  // the labels of four runs at a time
        uint32_t lb[4];
#pragma unroll
        for (int j = 0; j < 4; j++) lb[j] = lab[min(k + 4 * j, nblk - 1)];
#pragma unroll
        for (int j = 0; j < 4; j++) take(lb[j]);
    }
    if (zs) {
        zs = fill_up(m.conn, zs);
        if ((uint32_t)zs) atomicOr(&sz[lane][0], (uint32_t)zs);
        if (zs >> 32) atomicOr(&sz[lane][1], (uint32_t)(zs >> 32));
    }
    __syncthreads();
    if (oin) glb(out)[oi] = yz | (bw & twice32(sz[(w >> 1) * TBH + (p >> 1)][w & 1]));
    guard_report(gd, ok);
}

// ------------------------------------------------------------------ kernels
__device__ __forceinline__ void group_at(const CclGeo &q, int rows, int i, int &gx, int &ty) {
    const int n = ccl_groups_x(q, rows);
    ty = i / n;
    gx = i - ty * n;
}

// blockIdx.y: the labelling; the groups go to the XCDs in contiguous ranges
// (neighbouring groups share the cache lines of their mask rows)
template <int TBH, int NR, int NW, bool CANON>
__global__ __launch_bounds__(64 * NW) void k_ccl_local(Geo g, CclMulti m, int32_t *ncanon, int32_t *icanon) {
    const CclOp &o = m.op[blockIdx.y];
    const CclGeo q = ccl_geo(g, TBH);
    int gx, ty;
    group_at(q, NR, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), gx, ty);
    if (CANON && blockIdx.x == 0 && threadIdx.x < kCounterSlots && m.counters)
        for (int k = 0; k < 2; k++) glb(m.counters)[threadIdx.x * kCounterStep + k] = 0;
    ccl_local_group<TBH, NR, NW, CANON>(g, q, ccl_arrays(o.ws, g, q), o.b, o.y, o.z, o.multi, gx, ty, m.guard, ncanon, icanon);
}

__global__ __launch_bounds__(kThreads) void k_ccl_merge(Geo g, CclMulti m) {
    __shared__ int2 pairs[kThreads / 64][kMergePairs];
    const CclOp &o = m.op[blockIdx.y];
    const CclGeo q = ccl_geo(g, m.tbh);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int w = xcd_contiguous((int)blockIdx.x, (int)gridDim.x) * (kThreads / 64) + wv, tile = w >> 1;
    int unions = 0, tries = 0;
    if (tile < q.ntx * q.nty)
        ccl_merge_tile(g, q, ccl_arrays(o.ws, g, q), tile, w & 1, pairs[wv], unions, tries, m.guard);
    if (m.counters) {
        // one pair of additions per wave, spread over lines of their own (per
        // lane on one line they took most of this pass: 53 -> 11.8 us at 2048^2)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            unions += __shfl_xor(unions, off);
            tries += __shfl_xor(tries, off);
        }
        if (unions && lane_id() == 0) {
            unsigned long long *at = m.counters + w % kCounterSlots * kCounterStep;
            atomicAdd(&at[0], (unsigned long long)unions);
            atomicAdd(&at[1], (unsigned long long)(tries - unions));
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_ccl_flag(Geo g, CclMulti m) {
    const CclOp &o = m.op[blockIdx.y];
    const CclGeo q = ccl_geo(g, m.tbh);
    const int tile = (int)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (o.multi && tile < q.ntx * q.nty) ccl_flag_tile(q, ccl_arrays(o.ws, g, q), tile, m.guard);
}

template <int TBH>
__global__ __launch_bounds__(kThreads) void k_ccl_reseed(Geo g, CclMulti m) {
    const CclOp &o = m.op[blockIdx.y];
    const CclGeo q = ccl_geo(g, TBH);
    int gx, ty;
    group_at(q, 64, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), gx, ty);
    ccl_reseed_group<TBH>(g, q, ccl_arrays(o.ws, g, q), o.b, o.y, o.user, gx, ty, m.guard);
}

template <int TBH>
__global__ __launch_bounds__(kThreads) void k_ccl_gather(Geo g, CclMulti m) {
    const CclOp &o = m.op[blockIdx.y];
    const CclGeo q = ccl_geo(g, TBH);
    int gx, ty;
    group_at(q, 64, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), gx, ty);
    ccl_gather_group<TBH>(g, q, ccl_arrays(o.ws, g, q), o.b, o.y, o.z, o.user, o.multi, o.out, gx, ty, m.guard);
}

// Canonical labels: the smallest first pixel of each root's nodes, gathered at
// the root (one wave per tile).
__global__ __launch_bounds__(kThreads) void k_ccl_canon(Geo g, CclMulti m, int32_t *canon_) {
    const CclOp &o = m.op[0];
    const CclGeo q = ccl_geo(g, m.tbh);
    const int tile = (int)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (tile >= q.ntx * q.nty) return;
    const CclArrays a = ccl_arrays(o.ws, g, q);
    const VLG_GLOBAL int32_t *par = glb(a.par);
    VLG_GLOBAL int32_t *canon = glb(canon_);
    const int n = (int)glb(a.cnt)[tile], id0 = tile * q.np + 1, lane = lane_id();
    bool ok = true;
    for (int k0 = 0; k0 < n; k0 += 64) {
        const int id = id0 + k0 + lane;
        int r = id, v = 0, c = 0;
        if (k0 + lane < n) {
            v = canon[id];
            r = node_root(par, id, par[id], m.guard.cap, ok);
            if (r != id) c = __hip_atomic_load(&canon[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // one atomicMin for all of the wave's nodes of one root (a giant
        // component would otherwise serialise every wave on one address), none
        // where the root already holds a smaller index; after two roots every
        // lane by itself (a round trip per root of many small components)
        uint64_t pending = __ballot(r != id && v < c);
        for (int t = 0; t < 2 && pending; t++) {
            const int leader = __builtin_ctzll(pending);  // wave-uniform
            const int r0 = __builtin_amdgcn_readlane(r, leader);
            const bool mine = r == r0 && r != id;
            pending &= ~__ballot(mine);
            int least = mine ? v : 0x7fffffff;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) least = min(least, __shfl_xor(least, off));
            if (lane == leader && least < __hip_atomic_load(&canon[r0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                __hip_atomic_fetch_min(&canon[r0], least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (((pending >> lane) & 1) && v < __hip_atomic_load(&canon[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            __hip_atomic_fetch_min(&canon[r], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    guard_report(m.guard, ok);
}

// Canonical label of every pixel.  Runs look their label's value up into an
// LDS table by row and start; then a wave takes 16 of the 64 block rows, a
// lane per block, and writes the block's two pixels of each pixel row.
typedef int32_t lab2 __attribute__((ext_vector_type(2), aligned(4)));
template <int TBH>
__global__ __launch_bounds__(kThreads) void k_ccl_labels(Geo g, CclMulti m, const int32_t *ncanon_,
                                                         const int32_t *icanon_, int32_t *labels_) {
    using G = Grp<TBH, 64>;
    __shared__ uint64_t sb[G::PR * G::SBP];
    __shared__ RowMasks rm;
    __shared__ int V[kForest];
    __shared__ int snode[G::SUB * 2 * (64 + TBH)];  // canonical label of the tiles' nodes
    const CclOp &o = m.op[0];
    const CclGeo q = ccl_geo(g, TBH);
    const CclArrays a = ccl_arrays(o.ws, g, q);
    const VLG_GLOBAL int32_t *ncanon = glb(ncanon_), *icanon = glb(icanon_);
    VLG_GLOBAL int32_t *labels = glb(labels_);
    int gx, ty;
    group_at(q, 64, xcd_contiguous((int)blockIdx.x, (int)gridDim.x), gx, ty);
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    stage_rows<TBH>(g, o.b, gx, ty, tid, sb, rm);
    bool ok = true;
    {
        constexpr int TPS = kThreads / G::SUB;
        const int ns = tid / TPS, nx = gx * G::SUB + ns;
        if (nx < q.ntx) {
            const VLG_GLOBAL int32_t *par = glb(a.par);
            const int t = ty * q.ntx + nx, n = (int)glb(a.cnt)[t], id0 = t * q.np + 1;
            for (int j = tid % TPS; j < n; j += TPS)
                snode[ns * 2 * (64 + TBH) + j] = ncanon[node_root(par, id0 + j, par[id0 + j], m.guard.cap, ok)];
        }
    }
    __syncthreads();
    {
        const int sub = lane / TBH, rr = lane % TBH, tx = gx * G::SUB + sub, by = ty * TBH + rr;
        const Row r = rm.row(lane);
        const VLG_GLOBAL uint16_t *lab = glb(a.lab) + (int64_t)by * g.BW + tx * 64;
        int k = 0;
        for (uint64_t st = r.starts; st; st &= st - 1, k++) {
            if ((k & 3) != wave) continue;
            const uint32_t lb = lab[k];
            const int x = (int)(lb & 0x7FF);
            V[lane * 65 + __builtin_ctzll(st)] =
                lb & kLabNode ? snode[sub * 2 * (64 + TBH) + (int)(lb & 0xFF)]
                              : icanon[(int64_t)(ty * TBH + (x >> 6)) * g.BW + tx * 64 + (x & 63)];
        }
    }
    __syncthreads();
    for (int R = wave * 16; R < wave * 16 + 16; R++) {
        const int tx = gx * G::SUB + R / TBH, by = ty * TBH + R % TBH, bx = tx * 64 + lane, x = 2 * bx;
        if (by >= g.BH || tx >= q.ntx) continue;  // wave-uniform
        const Row r = rm.row(R);
        const int v = (r.fg() >> lane) & 1 ? V[R * 65 + run_of(r.starts, lane)] : -1;
#pragma unroll
        for (int d = 0; d < 2; d++) {
            const int yy = 2 * by + d;
            if (yy >= g.H || x >= g.W) continue;
            const int32_t v0 = ((d ? r.b0 : r.t0) >> lane) & 1 ? v : -1, v1 = ((d ? r.b1 : r.t1) >> lane) & 1 ? v : -1;
            VLG_GLOBAL int32_t *at = labels + (int64_t)yy * g.W + x;
            if (x + 1 < g.W) *(VLG_GLOBAL lab2 *)at = lab2{v0, v1};
            else at[0] = v0;
        }
    }
    guard_report(m.guard, ok);
}

// ---- batches (units: see kernels.hip)
template <int TBH>
__global__ __launch_bounds__(kThreads) void kb_ccl_local(BatchArgs a, BCcl o) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const CclGeo q = ccl_geo(d.g, TBH);
        int gx, ty;
        group_at(q, 64, (int)(u_ - a.prefix[ii]), gx, ty);
        ccl_local_group<TBH, 64, 4, false>(d.g, q, ccl_arrays(d.ws + d.off_ccl, d.g, q), bref(d, o.b), bref(d, o.y),
                                    bref(d, o.z), o.multi, gx, ty, a.guard, nullptr, nullptr);
        __syncthreads();  // the next group reuses the LDS
    }
}

__global__ __launch_bounds__(kThreads) void kb_ccl_merge(BatchArgs a, BCcl o) {
    __shared__ int2 pairs[kThreads / 64][kMergePairs];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int unions = 0, tries = 0;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const CclGeo q = ccl_geo(d.g, o.tbh);
        const int w = (int)(u_ - a.prefix[ii]) * (kThreads / 64) + wv, tile = w >> 1;
        if (tile < q.ntx * q.nty)
            ccl_merge_tile(d.g, q, ccl_arrays(d.ws + d.off_ccl, d.g, q), tile, w & 1, pairs[wv], unions, tries,
                           a.guard);
    }
}

__global__ __launch_bounds__(kThreads) void kb_ccl_flag(BatchArgs a, BCcl o) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const CclGeo q = ccl_geo(d.g, o.tbh);
        const int tile = (int)(u_ - a.prefix[ii]) * (kThreads / 64) +
                         __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        if (tile < q.ntx * q.nty) ccl_flag_tile(q, ccl_arrays(d.ws + d.off_ccl, d.g, q), tile, a.guard);
    }
}

template <int TBH>
__global__ __launch_bounds__(kThreads) void kb_ccl_reseed(BatchArgs a, BCcl o) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const CclGeo q = ccl_geo(d.g, TBH);
        int gx, ty;
        group_at(q, 64, (int)(u_ - a.prefix[ii]), gx, ty);
        ccl_reseed_group<TBH>(d.g, q, ccl_arrays(d.ws + d.off_ccl, d.g, q), bref(d, o.b), bref(d, o.y), o.user, gx,
                              ty, a.guard);
        __syncthreads();
    }
}

template <int TBH>
__global__ __launch_bounds__(kThreads) void kb_ccl_gather(BatchArgs a, BCcl o) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const CclGeo q = ccl_geo(d.g, TBH);
        int gx, ty;
        group_at(q, 64, (int)(u_ - a.prefix[ii]), gx, ty);
        ccl_gather_group<TBH>(d.g, q, ccl_arrays(d.ws + d.off_ccl, d.g, q), bref(d, o.b), bref(d, o.y), bref(d, o.z),
                              o.user, o.multi, bptr(d, o.out), gx, ty, a.guard);
        __syncthreads();
    }
}

#define VLG_BY_TBH(tbh, K)                   \
    switch (tbh) {                           \
    case 8: K(8); break;                     \
    case 16: K(16); break;                   \
    case 32: K(32); break;                   \
    default: return hipErrorInvalidValue;    \
    }

bool bad_multi(const CclMulti &m) { return m.n < 1 || m.n > kMaxMulti || !valid_tile_bh(m.tbh); }
dim3 group_grid(const Geo &g, const CclMulti &m, int rows) {
    const CclGeo q = ccl_geo(g, m.tbh);
    return dim3((unsigned)(ccl_groups_x(q, rows) * q.nty), (unsigned)m.n);
}
// Block rows and waves per group of the local pass.  Up to two groups of 64
// rows per compute unit the pass waits on its own chain of LDS round trips,
// which more waves shorten by sharing the columns; beyond that, the mask logic
// that every wave repeats fills the VALUs.  And while groups of 16 rows still
// find a compute unit each (64 groups of 64), they take a quarter of the
// columns per lane and a quarter of the unions per wave.  us, 64 rows and 4
// waves / 64 and 8 / 16 and 8: smoothed noise at 1024^2 (64 groups of 64 rows)
// 10.2 / 9.4 / 8.2, coin noise 20 / 16.0 / 10.1; at 1500^2 (141 groups)
// - / 9.6 / 11.7 and - / 16.3 / 15.2; smoothed noise at 4096^2 (1024 groups)
// 15.7 / 18.1 / -.  Tiles of 32 rows do not fit a group of 16.
enum class Split { few, some, many };  // 16 rows, 8 waves; 64 rows, 8 waves; 64 rows, 4 waves
Split local_split(const Geo &g, const CclMulti &m) {
    const CclGeo q = ccl_geo(g, m.tbh);
    const int64_t n = (int64_t)ccl_groups_x(q, 64) * q.nty * m.n;
    return m.tbh <= 16 && n <= 64 ? Split::few : n <= 512 ? Split::some : Split::many;
}
// per: waves per tile
dim3 tile_grid(const Geo &g, const CclMulti &m, int per) {
    const CclGeo q = ccl_geo(g, m.tbh);
    return dim3((unsigned)(((int64_t)per * q.ntx * q.nty + kThreads / 64 - 1) / (kThreads / 64)), (unsigned)m.n);
}
}  // namespace

hipError_t launch_ccl_local(hipStream_t s, const Geo &g, const CclMulti &m) {
    if (g.nwords == 0 || m.n == 0) return hipSuccess;
    if (bad_multi(m)) return hipErrorInvalidValue;
    const Split sp = local_split(g, m);
#define K(T)                                                                                             \
    if (sp == Split::few)                                                                                \
        k_ccl_local<T, T <= 16 ? 16 : 64, 8, false><<<group_grid(g, m, 16), 512, 0, s>>>(g, m, nullptr, nullptr); \
    else if (sp == Split::some)                                                                          \
        k_ccl_local<T, 64, 8, false><<<group_grid(g, m, 64), 512, 0, s>>>(g, m, nullptr, nullptr);       \
    else                                                                                                 \
        k_ccl_local<T, 64, 4, false><<<group_grid(g, m, 64), 256, 0, s>>>(g, m, nullptr, nullptr)
    VLG_BY_TBH(m.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_ccl_merge(hipStream_t s, const Geo &g, const CclMulti &m) {
    if (g.nwords == 0 || m.n == 0) return hipSuccess;
    if (bad_multi(m)) return hipErrorInvalidValue;
    if (ccl_geo(g, m.tbh).np == 0) return hipSuccess;  // one tile
    k_ccl_merge<<<tile_grid(g, m, 2), kThreads, 0, s>>>(g, m);
    return hipGetLastError();
}

hipError_t launch_ccl_flag(hipStream_t s, const Geo &g, const CclMulti &m) {
    bool any = false;
    for (int i = 0; i < m.n && i < kMaxMulti; i++) any |= m.op[i].multi != 0;
    if (g.nwords == 0 || !any) return hipSuccess;
    if (bad_multi(m)) return hipErrorInvalidValue;
    if (ccl_geo(g, m.tbh).np == 0) return hipSuccess;
    k_ccl_flag<<<tile_grid(g, m, 1), kThreads, 0, s>>>(g, m);
    return hipGetLastError();
}

hipError_t launch_ccl_reseed(hipStream_t s, const Geo &g, const CclMulti &m) {
    if (g.nwords == 0 || m.n == 0) return hipSuccess;
    if (bad_multi(m)) return hipErrorInvalidValue;
#define K(T) k_ccl_reseed<T><<<group_grid(g, m, 64), kThreads, 0, s>>>(g, m)
    VLG_BY_TBH(m.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_ccl_gather(hipStream_t s, const Geo &g, const CclMulti &m) {
    if (g.nwords == 0 || m.n == 0) return hipSuccess;
    if (bad_multi(m)) return hipErrorInvalidValue;
#define K(T) k_ccl_gather<T><<<group_grid(g, m, 64), kThreads, 0, s>>>(g, m)
    VLG_BY_TBH(m.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_ccl_labels(hipStream_t s, const Geo &g, const CclMulti &m, int32_t *ncanon, int32_t *icanon,
                             int32_t *labels) {
    if (g.nwords == 0) return hipSuccess;
    if (bad_multi(m) || m.n != 1) return hipErrorInvalidValue;
    const Split sp = local_split(g, m);
#define K(T)                                                                                             \
    if (sp == Split::few)                                                                                \
        k_ccl_local<T, T <= 16 ? 16 : 64, 8, true><<<group_grid(g, m, 16), 512, 0, s>>>(g, m, ncanon, icanon); \
    else if (sp == Split::some)                                                                          \
        k_ccl_local<T, 64, 8, true><<<group_grid(g, m, 64), 512, 0, s>>>(g, m, ncanon, icanon);          \
    else                                                                                                 \
        k_ccl_local<T, 64, 4, true><<<group_grid(g, m, 64), 256, 0, s>>>(g, m, ncanon, icanon)
    VLG_BY_TBH(m.tbh, K)
#undef K
    if (ccl_geo(g, m.tbh).np > 0) {
        k_ccl_merge<<<tile_grid(g, m, 2), kThreads, 0, s>>>(g, m);
        k_ccl_canon<<<tile_grid(g, m, 1), kThreads, 0, s>>>(g, m, ncanon);
    }
#define K(T) k_ccl_labels<T><<<group_grid(g, m, 64), kThreads, 0, s>>>(g, m, ncanon, icanon, labels)
    VLG_BY_TBH(m.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_b_ccl_local(hipStream_t s, const BatchArgs &a, int64_t total, const BCcl &o) {
    if (total == 0) return hipSuccess;
#define K(T) kb_ccl_local<T><<<persistent_grid(a, total), kThreads, 0, s>>>(a, o)
    VLG_BY_TBH(o.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_b_ccl_merge(hipStream_t s, const BatchArgs &a, int64_t total, const BCcl &o) {
    if (total == 0) return hipSuccess;
    if (!valid_tile_bh(o.tbh)) return hipErrorInvalidValue;
    kb_ccl_merge<<<persistent_grid(a, total), kThreads, 0, s>>>(a, o);
    return hipGetLastError();
}

hipError_t launch_b_ccl_flag(hipStream_t s, const BatchArgs &a, int64_t total, const BCcl &o) {
    if (total == 0 || !o.multi) return hipSuccess;
    if (!valid_tile_bh(o.tbh)) return hipErrorInvalidValue;
    kb_ccl_flag<<<persistent_grid(a, total), kThreads, 0, s>>>(a, o);
    return hipGetLastError();
}

hipError_t launch_b_ccl_reseed(hipStream_t s, const BatchArgs &a, int64_t total, const BCcl &o) {
    if (total == 0) return hipSuccess;
#define K(T) kb_ccl_reseed<T><<<persistent_grid(a, total), kThreads, 0, s>>>(a, o)
    VLG_BY_TBH(o.tbh, K)
#undef K
    return hipGetLastError();
}

hipError_t launch_b_ccl_gather(hipStream_t s, const BatchArgs &a, int64_t total, const BCcl &o) {
    if (total == 0) return hipSuccess;
#define K(T) kb_ccl_gather<T><<<persistent_grid(a, total), kThreads, 0, s>>>(a, o)
    VLG_BY_TBH(o.tbh, K)
#undef K
    return hipGetLastError();
}

}  // namespace vlg
