// vol.hip -- the logic on volumes (3-D images of D slices of H x W): N over
// the 26 voxels sharing a face, an edge or a vertex (the voxel included),
// and the labelling of 26-connected components behind reachability.
//
// A volume mask is D*H rows of packed words, slice after slice, exactly like
// a 2-D mask of D*H rows; only the spatial operators know the slices.  The
// labelling's union-find runs over the runs of 2 x 2 x 2 voxel blocks: any two
// voxels of such a block share a face, an edge or a vertex, so the foreground
// voxels of a block lie in one 26-component (the 3-D form of the 2 x 2 blocks
// of ccl.hip, whose run logic is shared, runs.h).
//
// Tiles of 8 x 8 block rows of 64 blocks (16 x 16 x 128 voxels), a lane per
// block row, labelled in LDS; then the contacts across tile borders are
// united in global memory.  The global forest is indexed by blocks, entries
// only for run starts and for a tile's last block column: par[id], id = block
// index + 1, 0 = "meets the seeds" (a labelling of one user), or flag bytes
// at the roots (several users).  256^3, five labellings with their gathers: 1950
// us with a lane per block and unions in global memory only (per labelling 223
// us unions, 76 seeds, 65 gather), 240 us now (local 25, merge 16, gather 7).
#include "runs.h"

namespace vlg {
namespace {

constexpr int kVlThreads = 256;
// The word of operand r at (slice z, row y, word w), complement applied,
// padding bits 0; 0 outside the volume.
__device__ __forceinline__ uint64_t vl_word(const Geo &g, int S, int D, const MRef &r, int z, int y, int w) {
    if (z < 0 || z >= D || y < 0 || y >= S || w < 0 || w >= g.wpr) return 0ull;
    const int64_t i = ((int64_t)z * S + y) * g.wpr + w;
    const uint64_t v = (r.p ? glb(r.p)[i] : 0ull) ^ r.inv;
    return w == g.wpr - 1 ? (v & g.tail) : v;
}

// N of operand x at word (z, y, w): the OR over the 3 x 3 rows (z+dz, y+dy)
// of each row dilated by one bit to each side.
__device__ __forceinline__ uint64_t vl_near_word(const Geo &g, int S, int D, const MRef &x, int z, int y, int w) {
    uint64_t n = 0;
#pragma unroll
    for (int dz = -1; dz <= 1; dz++) {
#pragma unroll
        for (int dy = -1; dy <= 1; dy++) {
            const uint64_t c = vl_word(g, S, D, x, z + dz, y + dy, w);
            const uint64_t l = vl_word(g, S, D, x, z + dz, y + dy, w - 1);
            const uint64_t h = vl_word(g, S, D, x, z + dz, y + dy, w + 1);
            n |= c | (c << 1) | (c >> 1) | (l >> 63) | (h << 63);
        }
    }
    return n;
}

// out = (N(x) ^ inv_out) OP z, one thread per word
__global__ __launch_bounds__(kVlThreads) void k_near3(Geo g, int S, int D, MRef x, uint64_t inv_out, MRef z, int zop,
                                                    uint64_t *out) {
    const int64_t wi = (int64_t)blockIdx.x * kVlThreads + threadIdx.x;
    if (wi >= g.nwords) return;
    const uint32_t row = fdiv((uint32_t)wi, g.wpr_mul, g.wpr_shift);
    const int w = (int)((uint32_t)wi - row * (uint32_t)g.wpr), zz = (int)row / S, y = (int)row - zz * S;
    const uint64_t n = vl_near_word(g, S, D, x, zz, y, w) ^ inv_out;
    const uint64_t zw = vl_word(g, S, D, z, zz, y, w);
    const uint64_t keep = w == g.wpr - 1 ? g.tail : ~0ull;
    glb(out)[wi] = (zop ? (n | zw) : (n & zw)) & keep;
}

// ------------------------------------------------------------------ labelling
constexpr int kV3Threads = 512, kV3Waves = kV3Threads / 64;
struct VlGeo {
    int S, D;
    int BX, BY, BZ;     // blocks
    int ntx, nty, ntz;  // tiles of 64 x 8 x 8 blocks
};
VlGeo vl_geo(const Geo &g, int S, int D) {
    VlGeo q{S, D, g.BW, (S + 1) / 2, (D + 1) / 2, 0, 0, 0};
    q.ntx = (q.BX + 63) / 64;
    q.nty = (q.BY + 7) / 8;
    q.ntz = (q.BZ + 7) / 8;
    return q;
}
struct VTile {
    int tx, ty, tz;
};
__device__ __forceinline__ VTile vl_tile(const VlGeo &q) {
    const int i = xcd_contiguous((int)blockIdx.x, (int)gridDim.x), yz = i / q.ntx;
    return VTile{i - yz * q.ntx, yz % q.nty, yz / q.nty};
}
// node id of block (bz, by, bx)
__device__ __forceinline__ int vl_id(const VlGeo &q, int bz, int by, int bx) { return (bz * q.BY + by) * q.BX + bx + 1; }

// Masks of N block rows: voxel row k>>1 (dz*2 + dy) of the block row, word k&1.
template <int N>
struct VMasks {
    uint32_t e[8][N], o[8][N];
    __device__ __forceinline__ void put(int k, int r, uint64_t w) { split_even_odd(w, e[k][r], o[k][r]); }
    __device__ __forceinline__ uint64_t even(int v, int r) const { return e[2 * v][r] | (uint64_t)e[2 * v + 1][r] << 32; }
    __device__ __forceinline__ uint64_t odd(int v, int r) const { return o[2 * v][r] | (uint64_t)o[2 * v + 1][r] << 32; }
};
// A block row: voxel (dz, dy, 0) and (dz, dy, 1) of its blocks, and its runs.
struct VRow {
    uint64_t e[4], o[4], conn, starts;
    __device__ __forceinline__ uint64_t fg() const { return starts | conn; }
};
template <int N>
__device__ __forceinline__ VRow vl_row(const VMasks<N> &m, int r) {
    VRow v;
    uint64_t l = 0, h = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        v.e[k] = m.even(k, r);
        v.o[k] = m.odd(k, r);
        l |= v.e[k];
        h |= v.o[k];
    }
    v.conn = l & (h << 1);
    v.starts = (l | h) & ~v.conn;
    return v;
}

// The four earlier neighbour block rows (oz, oy) of a block row, and the voxel
// rows (bit dz*2 + dy) in which a block touches them, on its side and theirs:
// two blocks at offset (oz, oy, ox) are 26-connected exactly when each has a
// voxel on the side facing the other.
constexpr int kRel = 4;
__device__ constexpr int kRelZ[kRel] = {0, -1, -1, -1}, kRelY[kRel] = {-1, -1, 0, 1};
__device__ constexpr uint32_t kRelMine[kRel] = {0x5, 0x1, 0x3, 0x2}, kRelTheirs[kRel] = {0xA, 0x8, 0xC, 0x4};

// Contacts of a row with an earlier one (blocks l with l, l-1, l+1), without
// those implied by another contact of the same two runs.
struct VContacts {
    uint64_t um, lm, rm;
};
__device__ __forceinline__ VContacts vl_contacts(uint64_t conn, uint64_t a0, uint64_t a1, uint64_t b0, uint64_t b1,
                                                 uint64_t uc) {
    const uint64_t u = (a0 | a1) & (b0 | b1), ul = a0 & (b1 << 1), ur = a1 & (b0 >> 1);
    return VContacts{u & ~(conn & ((uc & (u << 1)) | (ur << 1))), ul & ~((u & uc) | (conn & (u << 1))),
                     ur & ~(u & (uc >> 1))};
}
template <typename F>
__device__ __forceinline__ uint64_t vl_or(uint32_t rows, F f) {  // f(k) over the set bits of rows (a constant)
    uint64_t v = 0;
#pragma unroll
    for (int k = 0; k < 4; k++)
        if (rows >> k & 1) v |= f(k);
    return v;
}

// The tile's words of b: one per thread (16 slices x 16 rows x 2), returned.
struct VWord {
    int z, y, half;
    int64_t at;  // -1 outside the volume
};
__device__ __forceinline__ VWord vl_tile_word(const Geo &g, const VlGeo &q, const VTile &t, int tid) {
    VWord w{tid >> 5, (tid >> 1) & 15, tid & 1, -1};
    const int z = t.tz * 16 + w.z, y = t.ty * 16 + w.y, x = t.tx * 2 + w.half;
    if (z < q.D && y < q.S && x < g.wpr) w.at = ((int64_t)z * q.S + y) * g.wpr + x;
    return w;
}
__device__ __forceinline__ uint64_t vl_load(const Geo &g, const MRef &r, const VWord &w, int tx) {
    return w.at >= 0 ? ldm(r, w.at) & keep_of(g, tx * 2 + w.half) : 0ull;
}
// Masks of the tile's 64 block rows from its words staged in sb (16 x 16 x 3).
__device__ __forceinline__ uint64_t vl_split(const uint64_t *sb, VMasks<64> &m, int lane, int wave) {
    const int z = 2 * (lane >> 3) + (wave >> 2), y = 2 * (lane & 7) + ((wave >> 1) & 1);
    const uint64_t w = sb[(z * 16 + y) * 3 + (wave & 1)];
    m.put(wave, lane, w);
    return w;
}
constexpr int kVSb = 16 * 16 * 3, kVSa = 18 * 18 * 5;

// Words of y & z with a halo of one slice, row and word, into sa; and the
// blocks of voxel row and word `wave` that have a seed voxel, from them.
__device__ __forceinline__ void vl_stage_seeds(const Geo &g, const VlGeo &q, const VTile &t, const MRef &y,
                                               const MRef &z, int tid, uint64_t *sa) {
    constexpr int N = 18 * 18 * 4, IT = (N + kV3Threads - 1) / kV3Threads;
    uint64_t a[IT], b[IT];
    bool in[IT];
#pragma unroll
    for (int k = 0; k < IT; k++) {
        const int i = tid + k * kV3Threads, zz = t.tz * 16 + i / 72 - 1, yy = t.ty * 16 + (i >> 2) % 18 - 1,
                  ww = t.tx * 2 + (i & 3) - 1;
        in[k] = i < N && zz >= 0 && zz < q.D && yy >= 0 && yy < q.S && ww >= 0 && ww < g.wpr;
        const int64_t at = in[k] ? ((int64_t)zz * q.S + yy) * g.wpr + ww : 0;
        a[k] = y.p ? glb(y.p)[at] : 0ull;
        b[k] = z.p ? glb(z.p)[at] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < IT; k++) {
        const int i = tid + k * kV3Threads;
        if (i < N)
            sa[(i >> 2) * 5 + (i & 3)] =
                in[k] ? (a[k] ^ y.inv) & (b[k] ^ z.inv) & keep_of(g, t.tx * 2 + (i & 3) - 1) : 0ull;
    }
}
__device__ __forceinline__ uint32_t vl_seed_blocks(const uint64_t *sa, uint64_t bw, int lane, int wave) {
    const int z = 2 * (lane >> 3) + (wave >> 2), y = 2 * (lane & 7) + ((wave >> 1) & 1);
    uint64_t l = 0, c = 0, r = 0;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const uint64_t *s = sa + ((z + i) * 18 + y + j) * 5 + (wave & 1);
            l |= s[0];
            c |= s[1];
            r |= s[2];
        }
    const uint64_t n = (c | (c << 1) | (c >> 1) | (l >> 63) | (r << 63)) & bw;
    return even_bits(n | (n >> 1));
}
__device__ __forceinline__ uint64_t vl_seed_row(const uint32_t (*s)[64], int lane) {
    return (uint64_t)(s[0][lane] | s[2][lane] | s[4][lane] | s[6][lane]) |
           (uint64_t)(s[1][lane] | s[3][lane] | s[5][lane] | s[7][lane]) << 32;
}

// Components of a tile in LDS, as ccl_local_group (ccl.hip) with four earlier
// neighbour rows per row; wave w takes columns 8w .. 8w+7 of every row.
// CANON: canon[id] = the first voxel of every run.
template <bool CANON>
__global__ __launch_bounds__(kV3Threads) void k_v3_local(Geo g, VlGeo q, MRef b, MRef y, MRef z, int32_t *par_,
                                                         uint8_t *flag_, int multi, LoopGuard gd, int32_t *canon) {
    constexpr int CW = 64 / kV3Waves;
    __shared__ uint64_t sb[kVSb], sa[kVSa];
    __shared__ VMasks<64> vm;
    __shared__ uint32_t sseed[8][64];
    __shared__ uint64_t sconn[64], sstart[64];
    __shared__ int L[kForest];
    __shared__ uint32_t sbits[64][2];  // roots that meet the seeds
    __shared__ int pairs[kV3Waves][128];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
    const bool seeds = !multi && (y.p || y.inv) && (z.p || z.inv);
    {
        const VWord w = vl_tile_word(g, q, t, tid);
        const uint64_t v = vl_load(g, b, w, t.tx);
        if (seeds) vl_stage_seeds(g, q, t, y, z, tid, sa);
        sb[(w.z * 16 + w.y) * 3 + w.half] = v;
#pragma unroll
        for (int k = 0; k < (kForest + kV3Threads - 1) / kV3Threads; k++) {
            const int x = tid + k * kV3Threads;
            if (x < kForest) L[x] = x;
        }
        if (tid < 128) (&sbits[0][0])[tid] = 0;
    }
    __syncthreads();
    {
        const uint64_t bw = vl_split(sb, vm, lane, wave);
        if (seeds) sseed[wave][lane] = vl_seed_blocks(sa, bw, lane, wave);
    }
    __syncthreads();
    const VRow m = vl_row(vm, lane);
    if (wave == 0) {
        sconn[lane] = m.conn;
        sstart[lane] = m.starts;
    }
    __syncthreads();
    const int lz = lane >> 3, ly = lane & 7, bz = t.tz * 8 + lz, by = t.ty * 8 + ly;
    const Window<CW> win{CW * wave};
    const int row0 = lane * kRowStep, c0 = win.c0;
    const RunStarts sm = run_starts(win, m.starts);
    auto here = [&](int i) { return row0 + sm(c0 - 1, i); };  // this row's run at window bit i
    uint32_t um[kRel], lm[kRel], rm[kRel];
    RunStarts us[kRel];
    uint64_t has = 0;  // blocks of the runs that have a parent
#pragma unroll
    for (int r = 0; r < kRel; r++) {
        const bool in = (kRelZ[r] == 0 || lz > 0) && (kRelY[r] == 0 || (kRelY[r] < 0 ? ly > 0 : ly < 7));
        const int nl = in ? lane + 8 * kRelZ[r] + kRelY[r] : lane;
        const uint64_t a0 = vl_or(kRelMine[r], [&](int k) { return m.e[k]; }),
                       a1 = vl_or(kRelMine[r], [&](int k) { return m.o[k]; });
        const uint64_t b0 = in ? vl_or(kRelTheirs[r], [&](int k) { return vm.even(k, nl); }) : 0ull,
                       b1 = in ? vl_or(kRelTheirs[r], [&](int k) { return vm.odd(k, nl); }) : 0ull;
        us[r] = run_starts(win, sstart[nl]);
        const VContacts c = vl_contacts(m.conn, a0, a1, b0, b1, sconn[nl]);
        // the first contact of a run becomes its parent without a union
        const uint64_t all = c.um | c.lm | c.rm;
        const uint32_t f = win.own(all & ~(m.conn & (fill_up(m.conn, all) << 1)) & ~has);
        has |= fill_up(m.conn, starts_of(m.conn, all));
        um[r] = win.own(c.um);
        lm[r] = win.own(c.lm);
        rm[r] = win.own(c.rm);
        for (uint32_t x = f; x; x &= x - 1) {
            const int i = __builtin_ctz(x), off = (um[r] >> i) & 1 ? 0 : (lm[r] >> i) & 1 ? -1 : 1;
            L[here(i)] = nl * kRowStep + us[r](c0 - 1, i + off);
        }
        rm[r] &= ~(f & ~(um[r] | lm[r]));
        lm[r] &= ~(f & ~um[r]);
        um[r] &= ~f;
    }
    __syncthreads();
    bool ok = true;
    {
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
#pragma unroll
        for (int r = 0; r < kRel; r++) {
            const int nrow0 = row0 + (8 * kRelZ[r] + kRelY[r]) * kRowStep;
            for (;;) {
                const uint32_t x = um[r] | lm[r] | rm[r];
                const uint64_t act = __ballot(x != 0);
                if (!act) break;
                if (x) {
                    const int i = __builtin_ctz(x);
                    const uint32_t bit = x & (0u - x), isu = um[r] & bit, isl = isu | (lm[r] & bit);
                    const int at = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0u));
                    pairs[wave][at] = here(i) | (nrow0 + us[r](c0 - 1, i + (isu ? 0 : isl ? -1 : 1))) << 16;
                    um[r] &= ~bit;
                    if (!isu) lm[r] &= ~bit;
                    if (!isl) rm[r] &= ~bit;
                }
                n += __popcll(act);
                if (n >= 64) take(64);
            }
        }
        if (n > 0) take(n);
    }
    __syncthreads();
    // every run's root (two walks at a time), and the roots that meet the seeds
    const uint64_t ss = seeds ? starts_of(m.conn, vl_seed_row(sseed, lane)) : 0ull;
    const uint32_t ssw = win.of(ss);
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
            if ((ssw >> s[j]) & 1) atomicOr(&sbits[xr][xc >> 5], 1u << (xc & 31));
        }
    }
    __syncthreads();
    VLG_GLOBAL int32_t *par = glb(par_);
    auto id_of = [&](int v) {
        const int r = forest_row(v);
        return vl_id(q, t.tz * 8 + (r >> 3), t.ty * 8 + (r & 7), t.tx * 64 + v - r * kRowStep);
    };
    for (uint32_t st = sm.w & win.kOwn; st; st &= st - 1) {
        const int s = win.col(__builtin_ctz(st)), v = row0 + s, x = L[v], id = id_of(v);
        const bool seeded = x == v && ((sbits[lane][s >> 5] >> (s & 31)) & 1);
        par[id] = seeded ? 0 : id_of(x);
        if (multi) glb(flag_)[id] = 0;
        if (CANON) {
            // the run's first voxel: in its first voxel row that has one
            const uint64_t run = fill_up(m.conn, 1ull << s);
            int k = 0;
            while (k < 3 && !((m.e[k] | m.o[k]) & run)) k++;
            const uint64_t ev = k == 0 ? m.e[0] : k == 1 ? m.e[1] : k == 2 ? m.e[2] : m.e[3];
            const uint64_t od = k == 0 ? m.o[0] : k == 1 ? m.o[1] : k == 2 ? m.o[2] : m.o[3];
            const int l = __builtin_ctzll((ev | od) & run);
            const int xx = t.tx * 128 + 2 * l + ((ev >> l) & 1 ? 0 : 1);
            glb(canon)[id] = ((2 * bz + (k >> 1)) * q.S + 2 * by + (k & 1)) * g.W + xx;
        }
    }
    // the tile's last column has entries of its own: the tile to the right
    // touches it without knowing its run
    if (wave == kV3Waves - 1 && (m.conn >> 63)) {
        const int id = id_of(row0 + 63);
        par[id] = id_of(L[row0 + run_of(m.starts, 63)]);
        if (multi) glb(flag_)[id] = 0;
    }
    if (!multi && blockIdx.x == 0 && tid == 0) par[0] = 0;
    guard_report(gd, ok);
}

// Contacts across tile borders: the rows on a tile's border against the
// earlier rows in other tiles (columns shared by the waves), and the first and
// last column of every row against the tiles to the left and right.
constexpr int kExt = 9 * 10;  // block rows -1 .. 7 in z, -1 .. 8 in y
__global__ __launch_bounds__(kV3Threads) void k_v3_merge(Geo g, VlGeo q, MRef b, int32_t *par_, LoopGuard gd) {
    constexpr int CW = 64 / kV3Waves, N = 18 * 20 * 4;
    __shared__ uint64_t sb[18 * 20 * 5];
    __shared__ VMasks<kExt> vm;
    __shared__ uint32_t edge[kExt];  // bit k: voxel (k, x = 1) of block -1; bit 4 + k: voxel (k, x = 0) of block 64
    __shared__ int2 pairs[kV3Waves][128];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
#pragma unroll
    for (int k = 0; k < (N + kV3Threads - 1) / kV3Threads; k++) {
        const int i = tid + k * kV3Threads, zz = t.tz * 16 + i / 80 - 2, yy = t.ty * 16 + (i >> 2) % 20 - 2,
                  ww = t.tx * 2 + (i & 3) - 1;
        const bool in = i < N && zz >= 0 && zz < q.D && yy >= 0 && yy < q.S && ww >= 0 && ww < g.wpr;
        const uint64_t v = b.p ? glb(b.p)[in ? ((int64_t)zz * q.S + yy) * g.wpr + ww : 0] : 0ull;
        if (i < N) sb[(i >> 2) * 5 + (i & 3)] = in ? (v ^ b.inv) & keep_of(g, ww) : 0ull;
    }
    __syncthreads();
    for (int i = tid; i < 9 * kExt; i += kV3Threads) {
        const int r = i % kExt, k = i / kExt, z = 2 * (r / 10), y = 2 * (r % 10);
        if (k < 8) {
            vm.put(k, r, sb[((z + (k >> 2)) * 20 + y + ((k >> 1) & 1)) * 5 + 1 + (k & 1)]);
        } else {
            uint32_t e = 0;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const uint64_t *s = &sb[((z + (v >> 1)) * 20 + y + (v & 1)) * 5];
                e |= (uint32_t)(s[0] >> 63) << v | (uint32_t)(s[3] & 1) << (4 + v);
            }
            edge[r] = e;
        }
    }
    __syncthreads();
    const int lz = lane >> 3, ly = lane & 7, bz = t.tz * 8 + lz, by = t.ty * 8 + ly, me = (lz + 1) * 10 + ly + 1;
    const int row0 = vl_id(q, bz, by, t.tx * 64);  // id of the row's first block
    const VRow m = vl_row(vm, me);
    VLG_GLOBAL int32_t *par = glb(par_);
    bool ok = true;
    int n = 0;  // wave-uniform
    auto take = [&](int cnt) {
        wave_lds_handoff();
        n -= cnt;
        if (lane < cnt) {
            const int2 pr = pairs[wave][n + lane];
            g_unite<false>(par, pr.x, pr.y, gd.cap, ok);
        }
        wave_lds_handoff();
    };
    auto put = [&](bool has, int x, int y) {
        const uint64_t act = __ballot(has);
        if (has)
            pairs[wave][n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0u))] = make_int2(x, y);
        n += __popcll(act);
        if (n >= 64) take(64);
    };
    const uint64_t mine = below(CW) << (CW * wave);
#pragma unroll
    for (int r = 0; r < kRel; r++) {
        const bool cross = (kRelZ[r] < 0 && lz == 0) || (kRelY[r] < 0 && ly == 0) || (kRelY[r] > 0 && ly == 7);
        const int ne = me + 10 * kRelZ[r] + kRelY[r], nrow0 = row0 + (kRelZ[r] * q.BY + kRelY[r]) * q.BX;
        const uint64_t a0 = vl_or(kRelMine[r], [&](int k) { return m.e[k]; }),
                       a1 = vl_or(kRelMine[r], [&](int k) { return m.o[k]; });
        const VRow nb = vl_row(vm, ne);
        const uint64_t b0 = vl_or(kRelTheirs[r], [&](int k) { return nb.e[k]; }),
                       b1 = vl_or(kRelTheirs[r], [&](int k) { return nb.o[k]; });
        VContacts c = vl_contacts(m.conn, a0, a1, b0, b1, nb.conn);
        if (!cross) c = VContacts{0, 0, 0};
        auto list = [&](uint64_t x, int off) {
            x &= mine;
            while (__any(x != 0)) {
                const int l = x ? __builtin_ctzll(x) : 0;
                put(x != 0, row0 + run_of(m.starts, l), nrow0 + run_of(nb.starts, l + off));
                x &= x - 1;
            }
        };
        list(c.um, 0);
        list(c.lm, -1);
        list(c.rm, 1);
        // across the tile's sides (relation r by wave r)
        if (wave == r) {
            const uint32_t e = edge[ne];
            put((a0 & 1) && (e & kRelTheirs[r]), row0, nrow0 - 1);
            put((a1 >> 63) && (e >> 4 & kRelTheirs[r]), row0 + 63, nrow0 + 64);
        }
    }
    if (wave == kRel)  // the block to the left in the same row
        put(((m.e[0] | m.e[1] | m.e[2] | m.e[3]) & 1) && (edge[me] & 0xF), row0, row0 - 1);
    if (n > 0) take(n);
    guard_report(gd, ok);
}

// Several users of a labelling: flag the roots of the runs that meet the
// seeds, N(y & z) & b or (reseed) the mask y itself.
template <bool RESEED>
__global__ __launch_bounds__(kV3Threads) void k_v3_seed(Geo g, VlGeo q, MRef b, MRef y, MRef z, const int32_t *par_,
                                                        uint8_t *flag, uint32_t bit, LoopGuard gd) {
    __shared__ uint64_t sb[kVSb], sa[kVSa];
    __shared__ VMasks<64> vm, vs;
    __shared__ uint32_t sseed[8][64];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
    const VWord w = vl_tile_word(g, q, t, tid);
    sb[(w.z * 16 + w.y) * 3 + w.half] = vl_load(g, b, w, t.tx);
    if (RESEED) sa[(w.z * 16 + w.y) * 3 + w.half] = vl_load(g, y, w, t.tx);
    else vl_stage_seeds(g, q, t, y, z, tid, sa);
    __syncthreads();
    {
        const uint64_t bw = vl_split(sb, vm, lane, wave);
        if (RESEED) vl_split(sa, vs, lane, wave);
        else sseed[wave][lane] = vl_seed_blocks(sa, bw, lane, wave);
    }
    __syncthreads();
    const VRow m = vl_row(vm, lane);
    const uint64_t s = RESEED ? vl_row(vs, lane).fg() : vl_seed_row(sseed, lane);
    const int row0 = vl_id(q, t.tz * 8 + (lane >> 3), t.ty * 8 + (lane & 7), t.tx * 64);
    bool ok = true;
    uint64_t st = starts_of(m.conn, s);
    for (int k = 0; st; st &= st - 1, k++) {
        if ((k & (kV3Waves - 1)) != wave) continue;
        const int id = row0 + __builtin_ctzll(st);
        flag_or(glb(flag), node_root(glb(par_), id, glb(par_)[id], gd.cap, ok), bit);
    }
    guard_report(gd, ok);
}

// out = (y & z) | (voxels of b whose component meets the seeds)
__global__ __launch_bounds__(kV3Threads) void k_v3_gather(Geo g, VlGeo q, MRef b, MRef y, MRef z, const int32_t *par_,
                                                          const uint8_t *flag, int multi, uint32_t bit, uint64_t *out,
                                                          LoopGuard gd) {
    __shared__ uint64_t sb[kVSb];
    __shared__ VMasks<64> vm;
    __shared__ uint32_t sz[64][2];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
    const VWord w = vl_tile_word(g, q, t, tid);
    const uint64_t bw = vl_load(g, b, w, t.tx), yz = vl_load(g, y, w, t.tx) & vl_load(g, z, w, t.tx);
    sb[(w.z * 16 + w.y) * 3 + w.half] = bw;
    if (tid < 128) (&sz[0][0])[tid] = 0;
    __syncthreads();
    vl_split(sb, vm, lane, wave);
    __syncthreads();
    const VRow m = vl_row(vm, lane);
    const VLG_GLOBAL int32_t *par = glb(par_);
    const int row0 = vl_id(q, t.tz * 8 + (lane >> 3), t.ty * 8 + (lane & 7), t.tx * 64);
    bool ok = true;
    uint64_t zs = 0, st = m.starts;
    for (int k = 0; st; st &= st - 1, k++) {
        if ((k & (kV3Waves - 1)) != wave) continue;
        const int id = row0 + __builtin_ctzll(st);
        const int root = node_root(par, id, par[id], gd.cap, ok);
        if (multi ? (glb(flag)[root] & bit) != 0 : root == 0) zs |= st & (0 - st);
    }
    if (zs) {
        zs = fill_up(m.conn, zs);
        if ((uint32_t)zs) atomicOr(&sz[lane][0], (uint32_t)zs);
        if (zs >> 32) atomicOr(&sz[lane][1], (uint32_t)(zs >> 32));
    }
    __syncthreads();
    if (w.at >= 0) glb(out)[w.at] = yz | (bw & twice32(sz[(w.z >> 1) * 8 + (w.y >> 1)][w.half]));
    guard_report(gd, ok);
}

// Canonical labels: the smallest first voxel of a component's runs, gathered
// at its root.
__global__ __launch_bounds__(kV3Threads) void k_v3_canon(Geo g, VlGeo q, MRef b, const int32_t *par_, int32_t *canon_,
                                                         LoopGuard gd) {
    __shared__ uint64_t sb[kVSb];
    __shared__ VMasks<64> vm;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
    const VWord w = vl_tile_word(g, q, t, tid);
    sb[(w.z * 16 + w.y) * 3 + w.half] = vl_load(g, b, w, t.tx);
    __syncthreads();
    vl_split(sb, vm, lane, wave);
    __syncthreads();
    const VRow m = vl_row(vm, lane);
    const VLG_GLOBAL int32_t *par = glb(par_);
    VLG_GLOBAL int32_t *canon = glb(canon_);
    const int row0 = vl_id(q, t.tz * 8 + (lane >> 3), t.ty * 8 + (lane & 7), t.tx * 64);
    bool ok = true;
    // this wave's runs of each row, four at a time: their walks overlap
    uint64_t st = m.starts;
    for (int i = 0; i < wave; i++) st &= st - 1;
    while (__any(st != 0)) {
        int id[4], r[4], v[4], c[4];
        bool on[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            on[j] = st != 0;
            id[j] = r[j] = on[j] ? row0 + __builtin_ctzll(st) : row0;
            st = drop_bits<kV3Waves>(st);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = on[j] ? canon[id[j]] : 0;
#pragma unroll
        for (int j = 1; j < 4; j++)
            if (!on[j]) r[j] = r[0];
        if (on[0]) node_roots(par, r, gd.cap, ok);
#pragma unroll
        for (int j = 0; j < 4; j++) on[j] &= r[j] != id[j];
#pragma unroll
        for (int j = 3; j > 0; j--)  // neighbours of one root together
            if (on[j] && on[j - 1] && r[j] == r[j - 1]) {
                v[j - 1] = min(v[j - 1], v[j]);
                on[j] = false;
            }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            c[j] = on[j] ? __hip_atomic_load(&canon[r[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            // one atomicMin for all of the wave's runs of one root (a giant
            // component would otherwise serialise every wave on one address),
            // none where the root already holds a smaller index; after two
            // roots every lane by itself
            uint64_t pending = __ballot(on[j] && v[j] < c[j]);
            for (int t = 0; t < 2 && pending; t++) {
                const int leader = __builtin_ctzll(pending);  // wave-uniform
                const int r0 = __builtin_amdgcn_readlane(r[j], leader);
                const bool same = on[j] && r[j] == r0;
                pending &= ~__ballot(same);
                int least = same ? v[j] : 0x7fffffff;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) least = min(least, __shfl_xor(least, off));
                if (lane == leader && least < __hip_atomic_load(&canon[r0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    __hip_atomic_fetch_min(&canon[r0], least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if ((pending >> lane) & 1)
                __hip_atomic_fetch_min(&canon[r[j]], v[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    guard_report(gd, ok);
}

__global__ __launch_bounds__(kV3Threads) void k_v3_labels(Geo g, VlGeo q, MRef b, const int32_t *par_,
                                                          const int32_t *canon, int32_t *labels_, LoopGuard gd) {
    __shared__ uint64_t sb[kVSb];
    __shared__ VMasks<64> vm;
    __shared__ int V[kForest];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const VTile t = vl_tile(q);
    const VWord w = vl_tile_word(g, q, t, tid);
    sb[(w.z * 16 + w.y) * 3 + w.half] = vl_load(g, b, w, t.tx);
    __syncthreads();
    vl_split(sb, vm, lane, wave);
    __syncthreads();
    bool ok = true;
    {
        const VRow m = vl_row(vm, lane);
        const int row0 = vl_id(q, t.tz * 8 + (lane >> 3), t.ty * 8 + (lane & 7), t.tx * 64);
        uint64_t st = m.starts;
        for (int i = 0; i < wave; i++) st &= st - 1;
        while (st) {  // four runs at a time: their walks overlap
            int at[4], r[4];
            int n = 0;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                at[j] = st ? __builtin_ctzll(st) : at[0];
                n += st != 0;
                r[j] = row0 + at[j];
                st = drop_bits<kV3Waves>(st);
            }
            node_roots(glb(par_), r, gd.cap, ok);
            int v[4];
#pragma unroll
            for (int j = 0; j < 4; j++) v[j] = glb(canon)[r[j]];
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (j < n) V[lane * 65 + at[j]] = v[j];
        }
    }
    __syncthreads();
    typedef int32_t lab2 __attribute__((ext_vector_type(2), aligned(4)));
    for (int R = wave * 8; R < wave * 8 + 8; R++) {
        const VRow m = vl_row(vm, R);
        const int v = (m.fg() >> lane) & 1 ? V[R * 65 + run_of(m.starts, lane)] : -1;
        const int x = t.tx * 128 + 2 * lane;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int zz = t.tz * 16 + 2 * (R >> 3) + (k >> 1), yy = t.ty * 16 + 2 * (R & 7) + (k & 1);
            if (zz >= q.D || yy >= q.S || x >= g.W) continue;
            const int32_t v0 = (m.e[k] >> lane) & 1 ? v : -1, v1 = (m.o[k] >> lane) & 1 ? v : -1;
            VLG_GLOBAL int32_t *at = glb(labels_) + ((int64_t)zz * q.S + yy) * g.W + x;
            if (x + 1 < g.W) *(VLG_GLOBAL lab2 *)at = lab2{v0, v1};
            else at[0] = v0;
        }
    }
    guard_report(gd, ok);
}

// The labelling's arrays in its workspace of 5 bytes per block: parents (ids
// start at 1; entry 0, the seed node, only for one user) and, for several
// users, flag bytes behind them.
struct VlArrays {
    int32_t *par;
    uint8_t *flag;
};
VlArrays vl_arrays(void *ws, const VlGeo &q, int multi) {
    const size_t nb = (size_t)q.BX * q.BY * q.BZ;
    return VlArrays{(int32_t *)ws - (multi ? 1 : 0), (uint8_t *)ws + 4 * nb - 1};
}
unsigned vl_tiles(const VlGeo &q) { return (unsigned)(q.ntx * q.nty * q.ntz); }

}  // namespace

hipError_t launch_near3(hipStream_t s, const Geo &g, int S, int D, MRef x, int inv_out, MRef z, int zop,
                        uint64_t *out) {
    if (g.nwords == 0) return hipSuccess;
    if (S < 1 || D < 1 || (int64_t)S * D != g.H) return hipErrorInvalidValue;
    k_near3<<<(unsigned)((g.nwords + kVlThreads - 1) / kVlThreads), kVlThreads, 0, s>>>(
        g, S, D, x, inv_out ? ~0ull : 0ull, z, zop, out);
    return hipGetLastError();
}

int64_t vl_nblocks(const Geo &g, int S, int D) {
    const VlGeo q = vl_geo(g, S, D);
    return (int64_t)q.BX * q.BY * q.BZ;
}

bool vl_one_tile(const Geo &g, int S, int D) { return vl_tiles(vl_geo(g, S, D)) <= 1; }

hipError_t launch_vl_label(hipStream_t s, const Geo &g, int S, int D, const CclOp &o, const LoopGuard &gd) {
    if (g.nwords == 0) return hipSuccess;
    if (S < 1 || D < 1 || (int64_t)S * D != g.H) return hipErrorInvalidValue;
    const VlGeo q = vl_geo(g, S, D);
    const VlArrays a = vl_arrays(o.ws, q, o.multi);
    k_v3_local<false><<<vl_tiles(q), kV3Threads, 0, s>>>(g, q, o.b, o.y, o.z, a.par, a.flag, o.multi, gd, nullptr);
    if (vl_tiles(q) > 1) k_v3_merge<<<vl_tiles(q), kV3Threads, 0, s>>>(g, q, o.b, a.par, gd);
    if (o.multi) k_v3_seed<false><<<vl_tiles(q), kV3Threads, 0, s>>>(g, q, o.b, o.y, o.z, a.par, a.flag, 2u, gd);
    return hipGetLastError();
}

hipError_t launch_vl_reseed(hipStream_t s, const Geo &g, int S, int D, const CclOp &o, const LoopGuard &gd) {
    if (g.nwords == 0) return hipSuccess;
    const VlGeo q = vl_geo(g, S, D);
    const VlArrays a = vl_arrays(o.ws, q, o.multi);
    k_v3_seed<true><<<vl_tiles(q), kV3Threads, 0, s>>>(g, q, o.b, o.y, o.z, a.par, a.flag, 2u << o.user, gd);
    return hipGetLastError();
}

hipError_t launch_vl_gather(hipStream_t s, const Geo &g, int S, int D, const CclOp &o, const LoopGuard &gd) {
    if (g.nwords == 0) return hipSuccess;
    const VlGeo q = vl_geo(g, S, D);
    const VlArrays a = vl_arrays(o.ws, q, o.multi);
    k_v3_gather<<<vl_tiles(q), kV3Threads, 0, s>>>(g, q, o.b, o.y, o.z, a.par, a.flag, o.multi, 2u << o.user, o.out, gd);
    return hipGetLastError();
}

hipError_t launch_vl_labels(hipStream_t s, const Geo &g, int S, int D, MRef b, int *par, int *canon, int *labels,
                            const LoopGuard &gd) {
    if (g.nwords == 0) return hipSuccess;
    if (S < 1 || D < 1 || (int64_t)S * D != g.H) return hipErrorInvalidValue;
    const VlGeo q = vl_geo(g, S, D);
    const unsigned n = vl_tiles(q);
    const MRef none{nullptr, 0ull};
    k_v3_local<true><<<n, kV3Threads, 0, s>>>(g, q, b, none, none, par, nullptr, 0, gd, canon);
    if (n > 1) k_v3_merge<<<n, kV3Threads, 0, s>>>(g, q, b, par, gd);
    k_v3_canon<<<n, kV3Threads, 0, s>>>(g, q, b, par, canon, gd);
    k_v3_labels<<<n, kV3Threads, 0, s>>>(g, q, b, par, canon, labels, gd);
    return hipGetLastError();
}

}  // namespace vlg
