// kernels.hip -- HIP kernels for gfx950 (CDNA4, wave64) on 1-bit-packed masks.
//
// Operators (paper "A spatial model checker in GPU", Sect. 2): threshold
// atoms, pixel-wise Boolean connectives, N (Moore-neighbourhood dilation),
// and fused segments of the last two.  The reachability labelling is in
// ccl.hip, percentiles are in pct.hip.
//
// Every operator is written once as a per-unit device function; single-image
// kernels walk one image's units, batch kernels walk the units of many
// images of different sizes through per-image descriptors.
#include "dev.h"

#include <algorithm>

namespace vlg {
namespace {

// ------------------------------------------------------------------ Boolean
// out = ((x ^ x.inv) OP (y ^ y.inv)) ^ inv_out, OP = and (op 0) / or (op 1).
// A null operand is a constant (its inv); the loops below are specialised on
// that once per launch so that every load is unconditional and a thread keeps
// kLogicUnroll words in flight.
constexpr int kLogicUnroll = 4;

template <bool HX, bool HY, bool NT>
__device__ __forceinline__ void logic_span(const Geo &g, const uint64_t *__restrict__ xg, uint64_t xinv,
                                           const uint64_t *__restrict__ yg, uint64_t yinv, int op, uint64_t inv_out,
                                           uint64_t *__restrict__ outg, int64_t i0, int64_t stride, int64_t iend) {
    const VLG_GLOBAL uint64_t *xp = glb(xg), *yp = glb(yg);
    VLG_GLOBAL uint64_t *out = glb(outg);
    for (int64_t i = i0; i < iend; i += kLogicUnroll * stride) {
        uint64_t a[kLogicUnroll], b[kLogicUnroll];
#pragma unroll
        for (int k = 0; k < kLogicUnroll; k++) {
            const int64_t j = min(i + k * stride, iend - 1);
            a[k] = HX ? ld_hint<NT>(&xp[j]) ^ xinv : xinv;
            b[k] = HY ? ld_hint<NT>(&yp[j]) ^ yinv : yinv;
        }
#pragma unroll
        for (int k = 0; k < kLogicUnroll; k++) {
            const int64_t j = i + k * stride;
            uint64_t r = (op ? (a[k] | b[k]) : (a[k] & b[k])) ^ inv_out;
            if (is_last_col(g, j)) r &= g.tail;
            if (j < iend) out[j] = r;
        }
    }
}

// words i0, i0 + stride, ... below iend
template <bool NT = false>
__device__ __forceinline__ void logic_words(const Geo &g, const MRef &x, const MRef &y, int op, uint64_t inv_out,
                                            uint64_t *out, int64_t i0, int64_t stride, int64_t iend) {
    if (x.p && y.p) logic_span<true, true, NT>(g, x.p, x.inv, y.p, y.inv, op, inv_out, out, i0, stride, iend);
    else if (x.p) logic_span<true, false, NT>(g, x.p, x.inv, y.p, y.inv, op, inv_out, out, i0, stride, iend);
    else if (y.p) logic_span<false, true, NT>(g, x.p, x.inv, y.p, y.inv, op, inv_out, out, i0, stride, iend);
    else logic_span<false, false, NT>(g, x.p, x.inv, y.p, y.inv, op, inv_out, out, i0, stride, iend);
}

// ------------------------------------------------------------------ near
// out = (N(x) ^ inv_out) OP z, OP = and (zop 0) / or (zop 1).  N over the
// in-image 3x3 block, as a vertical sliding window: a lane owns a word column
// of a band of rows and walks down it, loading every row word once (the two
// edge lanes also load the word beyond the wave's edge), taking the left and
// right neighbour words from the adjacent lanes, and keeping the horizontally
// dilated rows y-1, y, y+1 in registers.  Each input word is fetched once per
// band instead of three times (by the workgroups of rows y-1, y, y+1, which
// sit on different XCDs with separate L2s).  The word columns of all bands are
// numbered in one sequence, 64 to a wave, so that the lanes of a wave are in
// use whatever the width: with one strip of a single band per wave, a batch of 128
// images of 128 to 2048 columns (2 to 32 words) took 46.5 us, 22.3 now.
// Complemented inputs have their padding bits cleared first so nothing leaks
// in from beyond the right border.
// Loads are issued unconditionally from clamped addresses and masked
// afterwards, so a chunk of CH rows has all its loads in flight at once.
// the band and the word column of this lane in a wave's task
__device__ __forceinline__ void near_column(const Geo &g, int64_t task, int R, int lane, bool &valid, int &band,
                                            int &w) {
    const uint32_t n = (uint32_t)((g.H + R - 1) / R) * (uint32_t)g.wpr, t = (uint32_t)task * 64u + (uint32_t)lane;
    valid = t < n;
    const uint32_t c = valid ? t : n - 1;
    band = (int)fdiv(c, g.wpr_mul, g.wpr_shift);
    w = (int)(c - (uint32_t)band * (uint32_t)g.wpr);
}
template <int CH, bool HZ>
__device__ __forceinline__ void near_band(const Geo &g, const uint64_t *__restrict__ xg, uint64_t xinv,
                                          uint64_t inv_out, const uint64_t *__restrict__ zg, uint64_t zinv, int zop,
                                          uint64_t *__restrict__ outg, int64_t task, int R) {
    const VLG_GLOBAL uint64_t *xp = glb(xg), *zp = glb(zg);
    VLG_GLOBAL uint64_t *out = glb(outg);
    const int lane = lane_id();
    bool valid;
    int band, wc;
    near_column(g, task, R, lane, valid, band, wc);
    const bool last = wc == g.wpr - 1;
    const int nb = lane == 0 ? wc - 1 : (lane == 63 ? wc + 1 : -1);  // word beyond the wave's edge
    const bool nbv = valid && nb >= 0 && nb < g.wpr;
    const int nbc = nbv ? nb : wc;
    const uint64_t keep = last ? g.tail : ~0ull;
    const int y0 = band * R, y1 = min(y0 + R, g.H);
    // raw loads of row y (clamped into the image) and their masking; the empty
    // asm consumes every raw value of a chunk after all its loads are issued,
    // which keeps the compiler from sinking a load into a conditional block
    // (with a wait right behind it)
    auto addr = [&](int y) { return (int64_t)min(max(y, 0), g.H - 1) * g.wpr; };
    auto mask_c = [&](int y, int lim, uint64_t raw) {
        return (y >= 0 && y <= lim && valid) ? ((raw ^ xinv) & keep) : 0ull;
    };
    auto mask_e = [&](int y, int lim, uint64_t raw) { return (y >= 0 && y <= lim && nbv) ? (raw ^ xinv) : 0ull; };
    // horizontal dilation of one row: the lanes beside may be of other bands
    // (all lanes take part)
    const uint64_t kl = wc > 0 ? ~0ull : 0ull, kr = last ? 0ull : ~0ull;
    auto hrow = [&](uint64_t c, uint64_t e) {
        uint64_t l = lane_prev64(c) & kl, r = lane_next64(c) & kr;
        if (lane == 0) l = e;
        if (lane == 63) r = e;
        return c | (c << 1) | (c >> 1) | (l >> 63) | (r << 63);
    };
    uint64_t hm, h0;
    {
        uint64_t rc0 = xp[addr(y0 - 1) + wc], re0 = xp[addr(y0 - 1) + nbc];
        uint64_t rc1 = xp[addr(y0) + wc], re1 = xp[addr(y0) + nbc];
        asm volatile("" : "+v"(rc0), "+v"(re0), "+v"(rc1), "+v"(re1));
        hm = hrow(mask_c(y0 - 1, g.H - 1, rc0), mask_e(y0 - 1, g.H - 1, re0));
        h0 = hrow(mask_c(y0, g.H - 1, rc1), mask_e(y0, g.H - 1, re1));
    }
    const int lim = min(y1, g.H - 1);
    for (int yb = y0; __any(yb < y1); yb += CH) {
        uint64_t c[CH], e[CH], zz[CH];
#pragma unroll
        for (int k = 0; k < CH; k++) {
            const int64_t a = addr(yb + 1 + k);
            c[k] = xp[a + wc];
            e[k] = xp[a + nbc];
            zz[k] = HZ ? zp[addr(yb + k) + wc] : 0ull;
        }
#pragma unroll
        for (int k = 0; k < CH; k++) {
            if (HZ) asm volatile("" : "+v"(c[k]), "+v"(e[k]), "+v"(zz[k]));
            else asm volatile("" : "+v"(c[k]), "+v"(e[k]));
        }
#pragma unroll
        for (int k = 0; k < CH; k++) {
            const uint64_t hp = hrow(mask_c(yb + 1 + k, lim, c[k]), mask_e(yb + 1 + k, lim, e[k]));
            const uint64_t n = (hm | h0 | hp) ^ inv_out;
            const uint64_t zv = HZ ? (zz[k] ^ zinv) : zinv;
            const uint64_t res = (zop ? (n | zv) : (n & zv)) & keep;
            if (valid && yb + k < y1) out[(int64_t)(yb + k) * g.wpr + wc] = res;
            hm = h0;
            h0 = hp;
        }
    }
}

// N of a constant mask (x.p == nullptr) is that constant over the image.
__device__ __forceinline__ void near_const_band(Geo g, uint64_t xinv, uint64_t inv_out, MRef z, int zop, uint64_t *out,
                                             int64_t task, int R) {
    bool valid;
    int band, w;
    near_column(g, task, R, lane_id(), valid, band, w);
    if (!valid) return;
    const uint64_t keep = w == g.wpr - 1 ? g.tail : ~0ull;
    const int y0 = band * R, y1 = min(y0 + R, g.H);
    for (int y = y0; y < y1; y++) {
        const int64_t i = (int64_t)y * g.wpr + w;
        const uint64_t n = xinv ^ inv_out, zz = ldm(z, i);
        out[i] = (zop ? (n | zz) : (n & zz)) & keep;
    }
}

// 64 word columns of bands of R (4, 8, 16 or 32) rows
__device__ __forceinline__ void near_task(const Geo &g, const MRef &x, uint64_t inv_out, const MRef &z, int zop,
                                          uint64_t *out, int64_t task, int R) {
    if (!x.p) near_const_band(g, x.inv, inv_out, z, zop, out, task, R);
    else if (R == 4 && z.p) near_band<4, true>(g, x.p, x.inv, inv_out, z.p, z.inv, zop, out, task, R);
    else if (R == 4) near_band<4, false>(g, x.p, x.inv, inv_out, z.p, z.inv, zop, out, task, R);
    else if (z.p) near_band<8, true>(g, x.p, x.inv, inv_out, z.p, z.inv, zop, out, task, R);
    else near_band<8, false>(g, x.p, x.inv, inv_out, z.p, z.inv, zop, out, task, R);
}

// ------------------------------------------------------------------ atoms
// The image is stored with a row pitch of wpr*64 elements, so mask word i
// covers elements [64 i, 64 i + 64) of a channel.  A wave takes 64
// consecutive words: lane l loads element 64 k + l for k = 0..63 (coalesced,
// all loads issued before any compare), then for each atom the wave-wide
// compare of pixel row k is the packed word k and is written into lane k's
// register (v_writelane).  One coalesced 512-byte store per atom.  The
// channel is read once for up to kMaxAtomsPerLaunch atoms.
// Four pixel rows per asm block: four compares write four SGPR pairs
// (s[84:91], reserved by the clobber list), then eight v_writelane move them
// into lanes k..k+3.  Each SGPR is read at least three VALU instructions
// after it was written and VCC is not involved, so the block needs no
// wait states of its own.
#define VLG_ATOM4(OP)                                                                               \
    asm(OP " s[84:85], %[a], %[t]\n\t" OP " s[86:87], %[b], %[t]\n\t" OP " s[88:89], %[c], %[t]\n\t" OP \
           " s[90:91], %[d], %[t]\n\t"                                                                 \
           "v_writelane_b32 %[lo], s84, %[k0]\n\tv_writelane_b32 %[hi], s85, %[k0]\n\t"                \
           "v_writelane_b32 %[lo], s86, %[k1]\n\tv_writelane_b32 %[hi], s87, %[k1]\n\t"                \
           "v_writelane_b32 %[lo], s88, %[k2]\n\tv_writelane_b32 %[hi], s89, %[k2]\n\t"                \
           "v_writelane_b32 %[lo], s90, %[k3]\n\tv_writelane_b32 %[hi], s91, %[k3]"                    \
        : [lo] "+v"(lo), [hi] "+v"(hi)                                                                \
        : [a] "v"(v[k]), [b] "v"(v[k + 1]), [c] "v"(v[k + 2]), [d] "v"(v[k + 3]), [t] "v"(t),       \
          [k0] "i"(k), [k1] "i"(k + 1), [k2] "i"(k + 2), [k3] "i"(k + 3)                             \
        : "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91")

template <int CMP, int NW>
__device__ __forceinline__ uint64_t atom_words(const float (&v)[NW], float t) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int k = 0; k < NW; k += 4) {
        if (CMP == 0) VLG_ATOM4("v_cmp_gt_f32_e64");
        else if (CMP == 1) VLG_ATOM4("v_cmp_lt_f32_e64");
        else if (CMP == 2) VLG_ATOM4("v_cmp_ge_f32_e64");
        else VLG_ATOM4("v_cmp_le_f32_e64");
    }
    return (uint64_t)lo | ((uint64_t)hi << 32);
}
#undef VLG_ATOM4

// One wave task: words [NW t, NW t + NW) of image channel img, for atoms
// 0..n-1 with thresholds sthr (LDS) and comparisons cmp; outf(j) is atom j's
// output mask.  NW = 64 (a full 512-byte store per atom) or, on images that
// would leave the chip idle, 16.
template <typename T, bool NT = false, int NW = 64, typename OutF>
__device__ __forceinline__ void atoms_task(const Geo &g, const T *__restrict__ img, int n, const uint8_t *cmp,
                                           const float *sthr, OutF outf, int64_t t) {
    const int lane = lane_id();
    const int64_t w0 = t * NW;
    const int nw = (int)((g.nwords - w0) < NW ? (g.nwords - w0) : NW);
    const VLG_GLOBAL T *src = glb(img) + w0 * 64 + lane;
    float v[NW];
    if (nw == NW) {
#pragma unroll
        for (int k = 0; k < NW; k++) v[k] = (float)ld_hint<NT>(&src[k * 64]);
    } else {
#pragma unroll
        for (int k = 0; k < NW; k++) v[k] = k < nw ? (float)ld_hint<NT>(&src[k * 64]) : 0.f;
    }
    const int64_t wi = w0 + lane;
    const uint64_t keep = (lane < nw && is_last_col(g, wi)) ? g.tail : ~0ull;
    for (int j = 0; j < n; j++) {
        const float th = sthr[j];
        uint64_t w;
        switch (cmp[j]) {
        case 0: w = atom_words<0, NW>(v, th); break;
        case 1: w = atom_words<1, NW>(v, th); break;
        case 2: w = atom_words<2, NW>(v, th); break;
        default: w = atom_words<3, NW>(v, th); break;
        }
        if (lane < nw) glb(outf(j))[wi] = w & keep;
    }
}

// ------------------------------------------------------------------ single-image kernels

template <bool NT>
__global__ __launch_bounds__(kThreads) void k_logic(Geo g, MRef x, MRef y, int op, uint64_t inv_out,
                                                    uint64_t *__restrict__ out) {
    logic_words<NT>(g, x, y, op, inv_out, out, (int64_t)blockIdx.x * kThreads + threadIdx.x,
                (int64_t)gridDim.x * kThreads, g.nwords);
}

__global__ __launch_bounds__(kThreads) void k_near(Geo g, MRef x, uint64_t inv_out, MRef z, int zop,
                                                   uint64_t *__restrict__ out, int R) {
    const int64_t ntasks = near_tasks(g, R), nwaves = (int64_t)gridDim.x * (kThreads / 64);
    for (int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); t < ntasks; t += nwaves)
        near_task(g, x, inv_out, z, zop, out, t, R);
}

// Up to kBatchMax independent Boolean steps (or near steps) in one launch:
// blockIdx.y selects the step.
template <bool NT>
__global__ __launch_bounds__(kThreads) void k_logic_batch(Geo g, LogicBatch bt) {
    const LogicOp &o = bt.ops[blockIdx.y];
    logic_words<NT>(g, o.x, o.y, o.op, o.inv_out, o.out, (int64_t)blockIdx.x * kThreads + threadIdx.x,
                (int64_t)gridDim.x * kThreads, g.nwords);
}

__global__ __launch_bounds__(kThreads) void k_near_batch(Geo g, NearBatch bt, int R) {
    const NearOp &o = bt.ops[blockIdx.y];
    const int64_t ntasks = near_tasks(g, R), nwaves = (int64_t)gridDim.x * (kThreads / 64);
    for (int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); t < ntasks; t += nwaves)
        near_task(g, o.x, o.inv_out, o.z, o.zop, o.out, t, R);
}

template <typename T, bool NT, int NW>
__global__ __launch_bounds__(kThreads) void k_atoms(Geo g, const T *__restrict__ img, AtomLaunch a) {
    __shared__ float sthr[kMaxAtomsPerLaunch];
    if ((int)threadIdx.x < a.n)
        sthr[threadIdx.x] = a.thr_dev[threadIdx.x] ? *a.thr_dev[threadIdx.x] : a.thr[threadIdx.x];
    __syncthreads();
    const int64_t nwaves = (int64_t)gridDim.x * (kThreads / 64);
    const int64_t ntasks = (g.nwords + NW - 1) / NW;
    auto outf = [&](int j) { return a.out[j]; };
    for (int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); t < ntasks; t += nwaves)
        atoms_task<T, NT, NW>(g, img, a.n, a.cmp, sthr, outf, t);
}

// Packed mask to one byte per pixel.  Bound by the stores: a thread writes 16
// consecutive output bytes, aligned to 16 whatever the width (a flat index
// over the image; only the unaligned head and tail and images narrower than
// 16 pixels go byte by byte).  7680^2: 74 us with one byte per thread, 11 us
// now (59 MB written, 5.4 TB/s).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t spread4(uint32_t n) {  // 4 bits to 4 bytes of 0 or 1
    return __umul24(n & 15u, 0x00204081u) & 0x01010101u;
}
// piece t of the image: bytes before the first aligned address (t = 0), then 16 each
__device__ __forceinline__ void unpack_piece(const Geo &g, const uint64_t *mask_, uint8_t *out_, int64_t t) {
    const VLG_GLOBAL uint64_t *mask = glb(mask_);
    VLG_GLOBAL uint8_t *out = glb(out_);
    const int64_t n = (int64_t)g.H * g.W;
    const int head = (int)(-(uintptr_t)out_ & 15);
    const int64_t i0 = t == 0 ? 0 : head + (t - 1) * 16;
    const int cnt = (int)min((int64_t)(t == 0 ? head : 16), n - i0);
    if (cnt <= 0) return;
    // (images hold fewer than 2^31 pixels)
    const uint32_t y = (uint32_t)i0 / (uint32_t)g.W, x = (uint32_t)i0 - y * (uint32_t)g.W;
    if (cnt == 16 && g.W >= 16) {
        // at most two rows; bits past a row's end are zero
        const int64_t w = (int64_t)y * g.wpr + (x >> 6);
        const int sh = x & 63, r = g.W - (int)x;
        uint64_t v = mask[w] >> sh;
        if (sh > 48 && (int)(x >> 6) + 1 < g.wpr) v |= mask[w + 1] << (64 - sh);
        if (r < 16) v |= mask[(int64_t)(y + 1) * g.wpr] << r;
        const uint32_t b = (uint32_t)v;
        *(VLG_GLOBAL u32x4_t *)(out + i0) = u32x4_t{spread4(b), spread4(b >> 4), spread4(b >> 8), spread4(b >> 12)};
    } else {
        uint32_t yy = y, xx = x;
        for (int k = 0; k < cnt; k++) {
            out[i0 + k] = (uint8_t)((mask[(int64_t)yy * g.wpr + (xx >> 6)] >> (xx & 63)) & 1);
            if (++xx == (uint32_t)g.W) {
                xx = 0;
                yy++;
            }
        }
    }
}
constexpr int kUnpackPieces = 4;  // pieces per thread of a batched unit
// pieces of an image: enough whatever the alignment of its output
__host__ __device__ inline int64_t unpack_pieces(const Geo &g) { return ((int64_t)g.H * g.W + 15) / 16 + 1; }

__global__ __launch_bounds__(kThreads) void k_unpack(Geo g, const uint64_t *mask, uint8_t *out) {
    unpack_piece(g, mask, out, (int64_t)blockIdx.x * kThreads + threadIdx.x);
}

// Rows of an image into its padded rows, the padding zero: 16 bytes of the
// destination per lane.  One launch and one pass instead of a fill and a
// pitched copy (loading 1000 x 750 uint16 pixels: 29.5 -> 18.8 us, launch bound).
__global__ __launch_bounds__(kThreads) void k_load_rows(const char *src, int64_t src_pitch, int64_t row_bytes,
                                                        uint32_t n, uint32_t mul, uint32_t shift, uint32_t pieces,
                                                        char *dst) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(1)));
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
        const uint32_t row = fdiv((uint32_t)i, mul, shift);
        const int64_t off = (int64_t)((uint32_t)i - row * pieces) * 16, left = row_bytes - off;
        const VLG_GLOBAL char *p = glb(src) + (int64_t)row * src_pitch + off;
        u4 v = {0u, 0u, 0u, 0u};
        if (left >= 16) {
            v = *(const VLG_GLOBAL u4u *)p;
        } else {
#pragma unroll
            for (int k = 0; k < 15; k++)
                if (k < left) v[k >> 2] |= (uint32_t)(uint8_t)p[k] << (8 * (k & 3));
        }
        *(VLG_GLOBAL u4 *)(glb(dst) + i * 16) = v;
    }
}

__global__ void k_fill_i64(unsigned long long *p, int n, unsigned long long v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ batch kernels
// Persistent: workgroup u-loop over the launch's global units.  Units per image:
//   BK_WORDS  256 mask words (atoms: four 64-word wave tasks)
//   BK_LOGIC  1024 mask words (Boolean steps)
//   BK_NEAR   256 word columns of bands (kBatchNearRows rows high, numbered
//             through all bands of the image, see near_band)
//   BK_TILES  one group of labelling tiles (64 block rows of tiles side by side)
//   BK_MERGE  two tiles (two waves each)  BK_FLAG   four tiles (one per wave)
//   BK_UNPACK 16384 output bytes
//   BK_PCTH   kPctUnit channel elements   BK_ONE    one per image

__global__ __launch_bounds__(kThreads) void kb_logic(BatchArgs a, BLogic ops) {
    const BLogicOp &o = ops.ops[blockIdx.y];
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const int64_t i0 = (u_ - a.prefix[ii]) * (kThreads * kLogicUnroll);
        const int64_t iend = min(i0 + kThreads * kLogicUnroll, d.g.nwords);
        logic_words(d.g, bref(d, o.x), bref(d, o.y), o.op, o.inv_out ? ~0ull : 0ull, bptr(d, o.out),
                    i0 + threadIdx.x, kThreads, iend);
    }
}

__global__ __launch_bounds__(kThreads) void kb_near(BatchArgs a, BNear ops) {
    const BNearOp &o = ops.ops[blockIdx.y];
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const int64_t t = (u_ - a.prefix[ii]) * (kThreads / 64) + (threadIdx.x >> 6);
        if (t < near_tasks(d.g, kBatchNearRows))
            near_task(d.g, bref(d, o.x), o.inv_out ? ~0ull : 0ull, bref(d, o.z), o.zop, bptr(d, o.out), t,
                      kBatchNearRows);
    }
}

template <typename T, bool NT>
__global__ __launch_bounds__(kThreads) void kb_atoms(BatchArgs a, BAtoms op) {
    __shared__ float sthr[kMaxAtomsPerLaunch];
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        __syncthreads();  // the previous unit is done with sthr
        if ((int)threadIdx.x < op.n) {
            const int p = op.pct[threadIdx.x];
            sthr[threadIdx.x] = p >= 0 ? glb((const float *)(d.ws + d.off_pct))[p] : op.thr[threadIdx.x];
        }
        __syncthreads();
        const T *img = (const T *)(d.img + (int64_t)op.chan * d.chan_bytes);
        const int64_t t = (u_ - a.prefix[ii]) * (kThreads / 64) + (threadIdx.x >> 6);
        auto outf = [&](int j) { return bptr(d, op.out[j]); };
        if (t * 64 < d.g.nwords) atoms_task<T, NT>(d.g, img, op.n, op.cmp, sthr, outf, t);
    }
}

// blockIdx.y: the output; dst[image * nout + output] (null: not wanted)
__global__ __launch_bounds__(kThreads) void kb_unpack(BatchArgs a, uint8_t *const *dst, int nout) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        uint8_t *out = glb(dst)[(int64_t)ii * nout + blockIdx.y];
        if (!out) continue;
        const uint64_t *mask = glb(d.outs)[blockIdx.y];
        const int64_t t0 = (u_ - a.prefix[ii]) * (kThreads * kUnpackPieces) + threadIdx.x;
        for (int k = 0; k < kUnpackPieces; k++) unpack_piece(d.g, mask, out, t0 + k * kThreads);
    }
}

#undef VLG_BATCH_LOOP
#undef VLG_BATCH_IMG

// ------------------------------------------------------------------ segments
// Instruction k as one scalar load of eight bytes (byte by byte it would be
// five vector loads, each waited for: most of a segment's time).
__device__ __forceinline__ SegIns seg_ins(const SegProg &p, int k) {
    uint64_t raw;
    __builtin_memcpy(&raw, &p.ins[k], sizeof raw);
    return SegIns{(uint8_t)raw, (uint8_t)(raw >> 8), (uint8_t)(raw >> 16), (uint8_t)(raw >> 24), (uint8_t)(raw >> 32)};
}

// Lane tiles: one wave (a workgroup of its own) per tile of one word column
// and 64 rows, the halo above and below included; lane l takes row r0 + l of
// every register as 128 bits, the column's word and 32 bits on each side.  The
// registers live in LDS, each lane reading and writing only its own entries,
// so no instruction needs a barrier; N takes the rows above and below from
// the adjacent lanes by DPP.  64 - 2 * halo rows are stored.  The window
// loses one bit per N at its ends and the edge lanes one row, all within the
// halo (at most 24).  Bound by the issue of one wave's instructions and, at
// 1024^2, half of the SIMDs without one: 9.3 us for a segment of 18 operators
// and halo 16 with three words per row and byte-wise instructions, 7.6 now.
//   LOAD    dst = ptr[a]
//   AND/OR  dst = ((a ^ ia) OP (b ^ ib)) ^ io
//   NEAR_*  dst = (N(a ^ ia) ^ io) OP (b ^ ib), N over the image's pixels only
//           (operand words outside the image and padding bits are background)
//   STORE   ptr[dst] = a ^ ia over the tile's centre (padding bits cleared)
struct SegRow {  // bits -32 .. 95 of the column
    uint32_t d[4];
};
__device__ __forceinline__ SegRow seg_row(uint64_t l, uint64_t c, uint64_t r) {
    return SegRow{{(uint32_t)(l >> 32), (uint32_t)c, (uint32_t)(c >> 32), (uint32_t)r}};
}
__global__ __launch_bounds__(64) void k_segment_lane(Geo g, SegProg p, int nty) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    extern __shared__ u4 lreg[];  // [register][lane]
    // each XCD takes a contiguous range of tiles, so the neighbour words and
    // halo rows that adjacent tiles load again come from that XCD's L2
    const int tile = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int lane = (int)threadIdx.x, TR = 64 - 2 * p.halo;
    const int tx = tile % g.wpr, ty = tile / g.wpr;
    const int row = ty * TR - p.halo + lane;
    const bool rin = row >= 0 && row < g.H;
    // the image's pixels in the window (background elsewhere)
    const uint64_t ml = rin && tx >= 1 ? ~0ull : 0ull;
    const uint64_t mc = rin ? (tx == g.wpr - 1 ? g.tail : ~0ull) : 0ull;
    const uint64_t mr = rin && tx + 1 < g.wpr ? (tx + 1 == g.wpr - 1 ? g.tail : ~0ull) : 0ull;
    const SegRow m = seg_row(ml, mc, mr);
    auto put = [&](int x, const SegRow &v) { lreg[x * 64 + lane] = u4{v.d[0], v.d[1], v.d[2], v.d[3]}; };
    auto get = [&](int x, uint32_t inv) {  // (kSegNone: the all-zero mask)
        const u4 v = x != kSegNone ? lreg[x * 64 + lane] : u4{0u, 0u, 0u, 0u};
        return SegRow{{v[0] ^ inv, v[1] ^ inv, v[2] ^ inv, v[3] ^ inv}};
    };
    // the leading loads, all in flight together
    int nl = 0;
    while (nl < p.nins && seg_ins(p, nl).op == SEG_LOAD) nl++;
    {
        const int64_t base = rin ? (int64_t)row * g.wpr + tx : 0;
        SegRow v[kSegMaxRegs];
#pragma unroll
        for (int j = 0; j < kSegMaxRegs; j++)
            if (j < nl) {
                const VLG_GLOBAL uint64_t *src = glb(p.ptr[seg_ins(p, j).a]);
                v[j] = seg_row(ml ? src[base - 1] : 0ull, rin ? src[base] : 0ull, mr ? src[base + 1] : 0ull);
            }
#pragma unroll
        for (int j = 0; j < kSegMaxRegs; j++)
            if (j < nl) put(seg_ins(p, j).dst, v[j]);
    }
    SegIns next = seg_ins(p, min(nl, kSegMaxIns - 1));
    for (int k = nl; k < p.nins; k++) {
        const SegIns in = next;
        next = seg_ins(p, min(k + 1, kSegMaxIns - 1));
        const uint32_t ia = (in.inv & 1) ? ~0u : 0u, ib = (in.inv & 2) ? ~0u : 0u, io = (in.inv & 4) ? ~0u : 0u;
        const SegRow a = get(in.a, ia);
        if (in.op == SEG_STORE) {
            if (lane >= p.halo && lane < p.halo + TR && rin) {
                const uint64_t v = (uint64_t)a.d[1] | (uint64_t)a.d[2] << 32;
                glb(p.ptr[in.dst])[(int64_t)row * g.wpr + tx] = tx == g.wpr - 1 ? (v & g.tail) : v;
            }
            continue;
        }
        const SegRow b = get(in.b, ib);
        SegRow r;
        if (in.op == SEG_AND || in.op == SEG_OR) {
            const bool o = in.op == SEG_OR;
#pragma unroll
            for (int w = 0; w < 4; w++) r.d[w] = (o ? a.d[w] | b.d[w] : a.d[w] & b.d[w]) ^ io;
        } else {
            // N over the image's pixels only
            uint32_t x[4], n[4];
#pragma unroll
            for (int w = 0; w < 4; w++) x[w] = a.d[w] & m.d[w];
#pragma unroll
            for (int w = 0; w < 4; w++) {
                const uint32_t lo = __builtin_amdgcn_alignbit(x[w], w > 0 ? x[w - 1] : 0u, 31),
                               hi = __builtin_amdgcn_alignbit(w < 3 ? x[w + 1] : 0u, x[w], 1);
                n[w] = x[w] | lo | hi;
            }
#pragma unroll
            for (int w = 0; w < 4; w++)
                n[w] = (n[w] | (uint32_t)lane_prev((int)n[w]) | (uint32_t)lane_next((int)n[w])) ^ io;
            const bool o = in.op == SEG_NEAR_OR;
#pragma unroll
            for (int w = 0; w < 4; w++) r.d[w] = o ? n[w] | b.d[w] : n[w] & b.d[w];
        }
        put(in.dst, r);
    }
}

// Wide tiles: an LDS row is 64 words (62 interior words and one halo word on
// each side), so lane l of every wave owns column l of the rows it is given
// (rows wave, wave + 8, ...); left and right neighbour words come from the
// adjacent lanes, the rows above and below from LDS.  Row r of register x is
// sreg[x * NI + r * 64 + lane].  Same instruction semantics as k_segment_lane.
constexpr int kSegWideThreads = 512;
constexpr int kSegWideWaves = kSegWideThreads / 64;
constexpr int kSegWideTW = 62;
__global__ __launch_bounds__(kSegWideThreads) void k_segment_wide(Geo g, SegProg p, int TR, int ntx) {
    extern __shared__ uint64_t sreg[];
    const int RR = TR + 2 * p.halo, NI = RR * 64;
    const int tx = (int)(blockIdx.x % ntx), ty = (int)(blockIdx.x / ntx);
    const int r0 = ty * TR - p.halo, w0 = tx * kSegWideTW - 1;
    const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
    const int w = w0 + lane;
    const bool win = w >= 0 && w < g.wpr;
    const uint64_t keep = w == g.wpr - 1 ? g.tail : ~0ull;
    int nl = 0;
    while (nl < p.nins && seg_ins(p, nl).op == SEG_LOAD) nl++;
    // the leading loads: for each input, all of this thread's rows in flight
    for (int j = 0; j < nl; j++) {
        const VLG_GLOBAL uint64_t *src = glb((const uint64_t *)p.ptr[seg_ins(p, j).a]);
        uint64_t *dst = sreg + seg_ins(p, j).dst * NI;
        for (int rb = wave; rb < RR; rb += kSegWideWaves * 8) {
            uint64_t v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int rr = rb + kSegWideWaves * u, row = r0 + rr;
                const bool in = win && rr < RR && row >= 0 && row < g.H;
                v[u] = in ? src[(int64_t)row * g.wpr + w] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int rr = rb + kSegWideWaves * u;
                if (rr < RR) dst[rr * 64 + lane] = v[u];
            }
        }
    }
    __syncthreads();
    for (int k = nl; k < p.nins; k++) {
        const SegIns in = seg_ins(p, k);
        const uint64_t ia = (in.inv & 1) ? ~0ull : 0ull, ib = (in.inv & 2) ? ~0ull : 0ull,
                       io = (in.inv & 4) ? ~0ull : 0ull;
        const uint64_t *A = in.a != kSegNone ? sreg + in.a * NI : nullptr;
        const uint64_t *B = in.b != kSegNone ? sreg + in.b * NI : nullptr;
        if (in.op == SEG_STORE) {
            // each thread stores the entries it owns (the same it writes in
            // every other instruction): no barrier needed before reuse
            VLG_GLOBAL uint64_t *out = glb(p.ptr[in.dst]);
            const bool col_ok = lane >= 1 && lane <= kSegWideTW && win;
            for (int rr = p.halo + wave; rr < p.halo + TR; rr += kSegWideWaves) {
                const int row = r0 + rr;
                if (!col_ok || row >= g.H) continue;
                out[(int64_t)row * g.wpr + w] = ((A ? A[rr * 64 + lane] : 0ull) ^ ia) & keep;
            }
            continue;
        }
        uint64_t *D = sreg + in.dst * NI;
        if (in.op == SEG_AND || in.op == SEG_OR) {
            for (int rr = wave; rr < RR; rr += kSegWideWaves) {
                const int i = rr * 64 + lane;
                const uint64_t x = (A ? A[i] : 0ull) ^ ia, y = (B ? B[i] : 0ull) ^ ib;
                D[i] = (in.op == SEG_OR ? (x | y) : (x & y)) ^ io;
            }
        } else {
            // N over the image's pixels only: rows and words outside the image
            // and padding bits count as background; rows outside the tile too
            // (they only reach the halo, which is inexact by design)
            auto hrow = [&](int r) -> uint64_t {
                const int row = r0 + r;
                const bool ok = win && r >= 0 && r < RR && row >= 0 && row < g.H;
                const uint64_t v = ok ? (((A ? A[r * 64 + lane] : 0ull) ^ ia) & keep) : 0ull;
                uint64_t l = __shfl_up(v, 1), h = __shfl_down(v, 1);
                if (lane == 0) l = 0ull;
                if (lane == 63) h = 0ull;
                return v | (v << 1) | (v >> 1) | (l >> 63) | (h << 63);
            };
            for (int rr = wave; rr < RR; rr += kSegWideWaves) {
                const uint64_t n = (hrow(rr - 1) | hrow(rr) | hrow(rr + 1)) ^ io;
                const int i = rr * 64 + lane;
                const uint64_t z = (B ? B[i] : 0ull) ^ ib;
                D[i] = in.op == SEG_NEAR_OR ? (n | z) : (n & z);
            }
        }
        __syncthreads();
    }
}


}  // namespace

// n / d = (umulhi(n, mul) + n) >> shift, valid for all 32-bit n
static void fast_div(uint32_t d, uint32_t &mul, uint32_t &shift) {
    uint32_t s = 0;
    while ((1ull << s) < d) s++;
    mul = (uint32_t)(((1ull << 32) * ((1ull << s) - d)) / d + 1);
    shift = s;
}

Geo make_geo(int H, int W) {
    Geo g;
    g.H = H;
    g.W = W;
    g.wpr = (W + 63) / 64;
    g.tail = (W % 64) ? ((1ull << (W % 64)) - 1) : ~0ull;
    g.nwords = (int64_t)H * g.wpr;
    g.BH = (H + 1) / 2;
    g.BW = (W + 1) / 2;
    fast_div((uint32_t)(g.wpr > 0 ? g.wpr : 1), g.wpr_mul, g.wpr_shift);
    return g;
}

hipError_t launch_load_rows(hipStream_t s, const void *src, int64_t src_pitch, int64_t row_bytes, int64_t rows,
                            void *dst, int64_t dst_pitch) {
    if (dst_pitch % 16 || row_bytes > dst_pitch || rows * (dst_pitch / 16) >= (1ll << 32))
        return hipErrorInvalidValue;
    uint32_t n = (uint32_t)(rows * (dst_pitch / 16));
    if (n == 0) return hipSuccess;
    uint32_t mul, shift;
    fast_div((uint32_t)(dst_pitch / 16), mul, shift);
    // (its own status: an error that the caller's thread left behind is not this launch's)
    uint32_t pieces = (uint32_t)(dst_pitch / 16);
    void *args[] = {&src, &src_pitch, &row_bytes, &n, &mul, &shift, &pieces, &dst};
    return hipLaunchKernel((const void *)k_load_rows, dim3(grid_for(n, kThreads, 16384)), dim3(kThreads), args, 0, s);
}

hipError_t launch_logic(hipStream_t s, const Geo &g, MRef x, MRef y, int op, int inv_out, uint64_t *out) {
    if (g.nwords == 0) return hipSuccess;
    const int grid = grid_for(g.nwords, kThreads, 4096);
    if (3 * g.nwords * 8 > kStreamBytes)
        k_logic<true><<<grid, kThreads, 0, s>>>(g, x, y, op, inv_out ? ~0ull : 0ull, out);
    else
        k_logic<false><<<grid, kThreads, 0, s>>>(g, x, y, op, inv_out ? ~0ull : 0ull, out);
    return hipGetLastError();
}

hipError_t launch_near(hipStream_t s, const Geo &g, MRef x, int inv_out, MRef z, int zop, uint64_t *out,
                       int rows) {
    if (g.nwords == 0) return hipSuccess;
    if (rows == 0) rows = near_band_rows(g);
    if (!valid_near_rows(rows)) return hipErrorInvalidValue;
    k_near<<<grid_for(near_tasks(g, rows), kThreads / 64, 8192), kThreads, 0, s>>>(g, x, inv_out ? ~0ull : 0ull, z,
                                                                                       zop, out, rows);
    return hipGetLastError();
}

template <typename T>
static hipError_t atoms_t(hipStream_t s, const Geo &g, const T *img, const AtomLaunch &a) {
    if (a.n < 1 || a.n > kMaxAtomsPerLaunch) return hipErrorInvalidValue;
    // tasks of 16 words while tasks of 64 would leave fewer than 2048 waves
    // (eight per compute unit): a 750 x 1000 uint16 image 13.0 -> 3.5 us, 24
    // evaluations of 256 to 3000 pixels a side 12.8 -> 9.1 us on average
    if (g.nwords < 2048 * 64) {
        k_atoms<T, false, 16><<<grid_for((g.nwords + 15) / 16, kThreads / 64, 8192), kThreads, 0, s>>>(g, img, a);
        return hipGetLastError();
    }
    const int grid = grid_for((g.nwords + 63) / 64, kThreads / 64, 8192);
    if (g.nwords * 64 * (int64_t)sizeof(T) + a.n * g.nwords * 8 > kStreamBytes)
        k_atoms<T, true, 64><<<grid, kThreads, 0, s>>>(g, img, a);
    else
        k_atoms<T, false, 64><<<grid, kThreads, 0, s>>>(g, img, a);
    return hipGetLastError();
}

hipError_t launch_atoms(hipStream_t s, const Geo &g, const void *chan, int dtype, const AtomLaunch &a) {
    if (g.nwords == 0) return hipSuccess;
    if (dtype == 1) return atoms_t(s, g, (const uint8_t *)chan, a);
    if (dtype == 2) return atoms_t(s, g, (const uint16_t *)chan, a);
    return atoms_t(s, g, (const float *)chan, a);
}

hipError_t launch_logic_batch(hipStream_t s, const Geo &g, const LogicBatch &b) {
    if (g.nwords == 0 || b.n == 0) return hipSuccess;
    dim3 grid(grid_for(g.nwords, kThreads, 4096), b.n);
    if (3 * b.n * g.nwords * 8 > kStreamBytes) k_logic_batch<true><<<grid, kThreads, 0, s>>>(g, b);
    else k_logic_batch<false><<<grid, kThreads, 0, s>>>(g, b);
    return hipGetLastError();
}

hipError_t launch_near_batch(hipStream_t s, const Geo &g, const NearBatch &b, int rows) {
    if (g.nwords == 0 || b.n == 0) return hipSuccess;
    if (rows == 0) rows = near_band_rows(g);
    if (!valid_near_rows(rows)) return hipErrorInvalidValue;
    dim3 grid(grid_for(near_tasks(g, rows), kThreads / 64, 8192), b.n);
    k_near_batch<<<grid, kThreads, 0, s>>>(g, b, rows);
    return hipGetLastError();
}

hipError_t launch_unpack(hipStream_t s, const Geo &g, const uint64_t *mask, uint8_t *out) {
    if (g.nwords == 0) return hipSuccess;
    k_unpack<<<(unsigned)((unpack_pieces(g) + kThreads - 1) / kThreads), kThreads, 0, s>>>(g, mask, out);
    return hipGetLastError();
}

// Tile of a segment: the shape with the least halo overhead among those that
// fit the LDS budget and leave at least kMinSegTiles tiles (or the most tiles
// when no shape leaves that many).  Wide tiles (62 words, k_segment_wide)
// count only the words of the image they cover.  When a narrow shape (1-16
// words) wins, the segment runs on lane tiles instead (k_segment_lane: one
// word column, 64 - 2 * halo rows per wave), which replaced narrow LDS tiles.
constexpr size_t kSegLdsBudget = 48 * 1024;
constexpr size_t kSegWideLdsBudget = 64 * 1024;
constexpr int64_t kMinSegTiles = 1024;
// lane tiles store at least 16 of their 64 rows
constexpr int kLaneSegMaxHalo = 24;
SegTile seg_tile(const Geo &g, int halo, int nregs) {
    SegTile best{4, 1, 0};
    double best_score = -1.0;
    auto consider = [&](int tr, int tw, size_t lds, double useful_w, int rw) {
        const int64_t tiles = (int64_t)((g.H + tr - 1) / tr) * ((g.wpr + tw - 1) / tw);
        const double eff = (double)tr * useful_w / ((double)(tr + 2 * halo) * rw);
        const double score = eff * std::min(1.0, (double)tiles / kMinSegTiles);
        if (score > best_score) {
            best_score = score;
            best = SegTile{tr, tw, lds};
        }
    };
    for (int tr : {4, 8, 16, 32, 64}) {
        const size_t lds = (size_t)nregs * (tr + 2 * halo) * 64 * 8;
        if (lds <= kSegWideLdsBudget) consider(tr, kSegWideTW, lds, std::min(kSegWideTW, g.wpr), 64);
    }
    for (int tw : {1, 2, 4, 8, 16}) {
        if (tw > 1 && tw / 2 >= g.wpr) break;
        for (int tr : {4, 8, 16, 32}) {
            const size_t lds = (size_t)nregs * (tr + 2 * halo) * (tw + 2) * 8;
            if (lds <= kSegLdsBudget) consider(tr, tw, lds, tw, tw + 2);
        }
    }
    if (best.lds_bytes == 0) best.lds_bytes = (size_t)nregs * (best.tr + 2 * halo) * (best.tw + 2) * 8;
    return best;
}

hipError_t launch_segment(hipStream_t s, const Geo &g, const SegProg &p) {
    if (g.nwords == 0) return hipSuccess;
    if (p.nins < 1 || p.nins > kSegMaxIns || p.nregs < 1 || p.nregs > kSegMaxRegs || p.halo < 0 || p.halo > 32)
        return hipErrorInvalidValue;
    const SegTile t = seg_tile(g, p.halo, p.nregs);
    const int ntx = (g.wpr + t.tw - 1) / t.tw, nty = (g.H + t.tr - 1) / t.tr;
    if (t.tw != kSegWideTW) {
        // lane tiles: one wave per word column and 64 - 2 * halo rows
        if (p.halo > kLaneSegMaxHalo) return hipErrorInvalidValue;
        const int lnty = (g.H + (64 - 2 * p.halo) - 1) / (64 - 2 * p.halo);
        const size_t lds = (size_t)p.nregs * 64 * 16;
        k_segment_lane<<<(int)((int64_t)g.wpr * lnty), 64, lds, s>>>(g, p, lnty);
    } else {
        if (t.lds_bytes > kSegWideLdsBudget) return hipErrorInvalidValue;
        k_segment_wide<<<ntx * nty, kSegWideThreads, t.lds_bytes, s>>>(g, p, t.tr, ntx);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ measurement
// Device-to-device copy for the HBM reference: each lane moves W-byte units
// (8 or 16) in a grid-stride loop with non-temporal loads and stores, so
// the copy streams past the caches like the large pixel-wise launches.
namespace {
template <typename T>
__global__ __launch_bounds__(kThreads) void k_stream_copy(const T *__restrict__ src, T *__restrict__ dst, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(glb(src) + i), glb(dst) + i);
}
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
}  // namespace

hipError_t launch_stream_copy(hipStream_t s, void *dst, const void *src, int64_t bytes, int width) {
    if (bytes <= 0) return hipSuccess;
    if ((width != 8 && width != 16) || bytes % width) return hipErrorInvalidValue;
    const int64_t n = bytes / width;
    const int grid = grid_for(n, kThreads, 256 * 64);
    if (width == 16)
        k_stream_copy<u32x4><<<grid, kThreads, 0, s>>>((const u32x4 *)src, (u32x4 *)dst, n);
    else
        k_stream_copy<uint64_t><<<grid, kThreads, 0, s>>>((const uint64_t *)src, (uint64_t *)dst, n);
    return hipGetLastError();
}

hipError_t launch_fill_i64(hipStream_t s, unsigned long long *p, int n, unsigned long long v) {
    k_fill_i64<<<(n + 255) / 256, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

// ------------------------------------------------------------------ batch launchers

int64_t batch_units(const Geo &g, int kind, int tbh) {
    if (g.nwords == 0) return 0;
    const CclGeo q = ccl_geo(g, tbh);
    const int64_t ntiles = (int64_t)q.ntx * q.nty;
    switch (kind) {
    case BK_WORDS: return (g.nwords + kThreads - 1) / kThreads;
    case BK_LOGIC: return (g.nwords + kThreads * kLogicUnroll - 1) / (kThreads * kLogicUnroll);
    case BK_NEAR: return (near_tasks(g, kBatchNearRows) + kThreads / 64 - 1) / (kThreads / 64);
    case BK_TILES: return (int64_t)ccl_groups_x(q, 64) * q.nty;
    case BK_MERGE: return (2 * ntiles + kThreads / 64 - 1) / (kThreads / 64);
    case BK_FLAG: return (ntiles + kThreads / 64 - 1) / (kThreads / 64);
    case BK_UNPACK: return (unpack_pieces(g) + kThreads * kUnpackPieces - 1) / (kThreads * kUnpackPieces);
    case BK_PCTH: return ((int64_t)g.H * g.wpr * 64 + kPctUnit - 1) / kPctUnit;
    case BK_ONE: return 1;
    }
    return 0;
}

hipError_t launch_b_atoms(hipStream_t s, const BatchArgs &a, int64_t total, const BAtoms &op) {
    if (total == 0) return hipSuccess;
    if (op.n < 1 || op.n > kMaxAtomsPerLaunch) return hipErrorInvalidValue;
    // a unit is 256 words: 16384 channel elements in, 256 words out per atom
    const int64_t bytes = total * (16384 * (a.dtype == 1 ? 1 : a.dtype == 2 ? 2 : 4) + op.n * 256 * 8);
    const int grid = persistent_grid(a, total);
    if (a.dtype == 1) {
        if (bytes > kStreamBytes) kb_atoms<uint8_t, true><<<grid, kThreads, 0, s>>>(a, op);
        else kb_atoms<uint8_t, false><<<grid, kThreads, 0, s>>>(a, op);
    } else if (a.dtype == 2) {
        if (bytes > kStreamBytes) kb_atoms<uint16_t, true><<<grid, kThreads, 0, s>>>(a, op);
        else kb_atoms<uint16_t, false><<<grid, kThreads, 0, s>>>(a, op);
    } else {
        if (bytes > kStreamBytes) kb_atoms<float, true><<<grid, kThreads, 0, s>>>(a, op);
        else kb_atoms<float, false><<<grid, kThreads, 0, s>>>(a, op);
    }
    return hipGetLastError();
}

hipError_t launch_b_unpack(hipStream_t s, const BatchArgs &a, int64_t total, uint8_t *const *dst, int nout) {
    if (total == 0 || nout == 0) return hipSuccess;
    kb_unpack<<<dim3(persistent_grid(a, total), nout), kThreads, 0, s>>>(a, dst, nout);
    return hipGetLastError();
}

hipError_t launch_b_logic(hipStream_t s, const BatchArgs &a, int64_t total, const BLogic &op) {
    if (total == 0 || op.n == 0) return hipSuccess;
    dim3 grid(persistent_grid(a, total), op.n);
    kb_logic<<<grid, kThreads, 0, s>>>(a, op);
    return hipGetLastError();
}

hipError_t launch_b_near(hipStream_t s, const BatchArgs &a, int64_t total, const BNear &op) {
    if (total == 0 || op.n == 0) return hipSuccess;
    dim3 grid(persistent_grid(a, total), op.n);
    kb_near<<<grid, kThreads, 0, s>>>(a, op);
    return hipGetLastError();
}

}  // namespace vlg
