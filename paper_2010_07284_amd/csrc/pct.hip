// pct.hip -- percentiles: the k-th smallest value of a channel (nearest rank,
// paper Sect. 3, threshold atoms against a percentile), up to four ranks of
// one channel together.
//
// Keys are the float32 bit patterns made order-preserving (negatives
// complemented, positives with the sign bit set) or the integer values.
//
// Sampled select (float32 and uint16): one workgroup takes 16384 samples and
// brackets every rank between two sample keys, five standard deviations of
// the sampling wide; one pass over the channel counts the keys below each
// bracket and collects those inside (1 to 4% of the channel per rank); the
// rank's key is then found among the collected ones.  Exact: when the bracket
// missed its rank, or too many keys fell inside, the same launches go over the
// whole channel instead.  A bracket that one value fills (a constant
// background) counts that value instead of collecting it.
// It reads the channel once where a radix select reads it three times (uint16:
// twice).  One rank of a 4096^2 float32 channel: 109 -> 52 us (the pass itself
// 16 us, 4.1 TB/s); three ranks of 128 images of 0.16 Gpixel: 585 -> 320 us
// (the pass 186 us, 3.5 TB/s, the gather of samples 43 us).
//
// Radix select (uint8, one pass; four ranks of a large uint16 channel; plans
// without room for candidates): each pass histograms one digit of the keys that
// agree with the digits chosen so far, then one workgroup finds the bucket
// holding the rank.
#include "dev.h"

namespace vlg {
namespace {

__device__ __forceinline__ uint32_t f32_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_f32(uint32_t k) {
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}

template <typename T> struct Vec4;
template <> struct Vec4<float> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct Vec4<uint8_t> { typedef uint8_t type __attribute__((ext_vector_type(4))); };
template <> struct Vec4<uint16_t> { typedef uint16_t type __attribute__((ext_vector_type(4))); };

template <typename T>
__device__ __forceinline__ uint32_t key_of(T v) {
    if constexpr (sizeof(T) == 4) return f32_key(v);
    else return (uint32_t)v;
}
template <typename T>
__device__ __forceinline__ float value_of(uint32_t k) {
    if constexpr (sizeof(T) == 4) return key_f32(k);
    else return (float)k;
}
// The largest key of an open bracket: uint16 keys end there; the largest
// float32 key stands for no element in the pass.  Brackets are no wider than
// the keys, so uint16 candidates have two digits (11 bits, 5) and only float32
// ones a third.
template <bool F32>
constexpr uint32_t kTopKey = F32 ? 0xFFFFFFFEu : 0xFFFFu;

// ------------------------------------------------------------------ sampled select
constexpr int kSelThreads = 1024;
// Samples: each costs a cache line of its own, so fewer of them on smaller
// images (16384 of a 1.25 Mpixel image would read 40% of it).  Their keys have
// to fit the candidates' room, pixels / 16 for each of four ranks, and so have
// the bracketed keys: 4.6% of the channel at the median with 12288 samples.
constexpr int kSample = 16384;
// Up to here one workgroup selects over the whole channel (65536 pixels take
// it over 40 us: its first digits collide).
constexpr int kDirectPixels = 32768;
__host__ __device__ inline uint32_t samples_of(uint32_t n) {
    return n < 131072u ? kSample / 2 : n < 2u << 20 ? kSample / 4 * 3 : kSample;
}
constexpr int kSegs = 16;        // candidate segments of a large single image (see PctSeg)
constexpr int kFewCandidates = 65536;  // one workgroup picks among these by itself
constexpr int kList = 4096;

// LIGHT: candidates are the keys in [lo, hi].  HEAVY (ties): those in (lo, hi),
// with the keys equal to lo and hi counted.  DIRECT: select over the channel.
enum PctMode : uint32_t { PCT_LIGHT = 0, PCT_HEAVY, PCT_DIRECT };
// Counts of the pass.  The workgroups of a large single image would all add to
// the same four addresses when they end (2048 of them: 40 us), so they share
// kSegs sets of counts and candidate segments, each on a cache line of its
// own.  A workgroup starts with the segment that a hash of its index names, its
// waves go round the segments whenever their queues are full, and what is left
// of them at its end passes a full segment by: with the index modulo kSegs the
// segment followed the rows, and an image periodic over 8 to 256 rows filled a
// few segments and left the others empty.
struct PctSeg {
    // ncand: places asked for, also beyond the segment's room; lost: candidates
    // (of several segments) that found no room
    uint32_t ncand, below, eqlo, eqhi, lost, pad[27];
};
struct PctQ {  // of one rank
    uint32_t k, lo, hi, mode;
    uint32_t nlist;
    uint32_t ties;  // the sample holds an end of the bracket kTies times or more
    uint32_t pad[26];
    PctSeg seg[kSegs];
    uint32_t hist[2048];   // of the candidates' leading digit
    // candidates in the rank's bucket of hist (nlist of them), or, when there
    // are too many (nlist = kCrowded), the histograms of the next two digits
    uint32_t list[kList];
};
constexpr uint32_t kCrowded = ~0u;
constexpr uint32_t kTies = 8;
static_assert(sizeof(PctQ) <= kPctStateBytes, "percentile state");
__device__ __forceinline__ VLG_GLOBAL PctQ *qstate(void *states, int slot) {
    return (VLG_GLOBAL PctQ *)((char *)states + (size_t)slot * kPctStateBytes);
}
// candidates of rank j: nseg segments of cap / nseg keys at buf + j * cap
struct Cand {
    uint32_t *buf;
    uint32_t cap;
    int nseg;
    __device__ __forceinline__ uint32_t seg_cap() const { return cap / (uint32_t)nseg; }
    __device__ __forceinline__ VLG_GLOBAL uint32_t *rank(int j) const { return glb(buf) + (size_t)j * cap; }
    // Places for n keys in segment s: how many it has room for, from its place `at` on.
    __device__ __forceinline__ uint32_t reserve(VLG_GLOBAL PctQ *st, int s, uint32_t n, uint32_t &at) const {
        at = __hip_atomic_fetch_add(&st->seg[s].ncand, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return at < seg_cap() ? min(n, seg_cap() - at) : 0u;
    }
};
__host__ __device__ inline uint32_t pixels_of(const Geo &g) { return (uint32_t)g.H * (uint32_t)g.W; }

// h[bin] += 1 for every active lane; many lanes with the first lane's bin add
// once together (a constant background would otherwise serialise the wave: two
// ranks at 4096^2 with 58% zeros 173 -> 139 us; without ties 113 -> 117).
__device__ __forceinline__ void hist_add(uint32_t *h, uint32_t bin) {
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    const uint64_t same = __ballot(bin == b);
    if (__popcll(same) > 8) {
        if (lane_id() == __builtin_ctzll(same)) atomicAdd(&h[b], (uint32_t)__popcll(same));
        if (bin == b) return;
    }
    atomicAdd(&h[bin], 1u);
}

// Bucket of rank r in a histogram of 2048 bins in LDS, by one wave; r becomes
// the rank inside the bucket (both wave-uniform).
__device__ __forceinline__ int wave_find(const uint32_t *h, uint32_t &r) {
    constexpr int PER = 32;
    const int lane = lane_id();
    uint32_t sum = 0;
#pragma unroll 8
    for (int j = 0; j < PER; j++) sum += h[lane * PER + ((j + lane) & (PER - 1))];  // (rotated: no bank conflicts)
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(inc, d);
        if (lane >= d) inc += t;
    }
    const uint64_t past = __ballot(inc > r);
    const int l = past ? __builtin_ctzll(past) : 63;
    r -= __builtin_amdgcn_readlane((int)inc, l) - __builtin_amdgcn_readlane((int)sum, l);
    // the bucket's lane owns 32 bins: again, a bin per lane
    const uint32_t c = lane < PER ? h[l * PER + lane] : 0u;
    inc = c;
#pragma unroll
    for (int d = 1; d < PER; d <<= 1) {
        const uint32_t t = __shfl_up(inc, d);
        if (lane >= d) inc += t;
    }
    const uint64_t p2 = __ballot(inc > r) & 0xFFFFFFFFull;
    const int m = p2 ? __builtin_ctzll(p2) : PER - 1;
    r -= __builtin_amdgcn_readlane((int)inc, m) - __builtin_amdgcn_readlane((int)c, m);
    return l * PER + m;
}

// The sample's ranks that bracket rank k of n: five standard deviations of
// the sample's rank of that value to each side.
__device__ __forceinline__ void sample_ranks(uint32_t k, uint32_t n, uint32_t sn, int &lo, int &hi) {
    const float q = ((float)k + 0.5f) / (float)n, c = q * (float)sn;
    const float d = 5.f * sqrtf((float)sn * q * (1.f - q)) + 3.f;
    lo = (int)floorf(c - d);
    hi = (int)ceilf(c + d);
}

// The i-th sample's key: one pixel of the i-th of sn equal parts, at a hashed
// place.  Gathered by many workgroups: a load touches a cache line of its
// own, and one compute unit has too few of them in flight (31 us for 16384).
template <typename T>
__device__ __forceinline__ void pct_gather(const Geo &g, const T *img, const Cand &cand, uint32_t i) {
    const uint32_t n = pixels_of(g), sn = samples_of(n);
    if (n <= kDirectPixels || i >= sn) return;
    const uint32_t a = (uint32_t)(((uint64_t)i * n) / sn), b = (uint32_t)(((uint64_t)(i + 1) * n) / sn);
    uint32_t x = i * 0x9E3779B1u;
    x = (x ^ (x >> 15)) * 0x85EBCA77u;
    const uint32_t p = a + __umulhi(x ^ (x >> 13), b - a), y = p / (uint32_t)g.W;
    glb(cand.buf)[i] = key_of<T>(glb(img)[(int64_t)y * g.wpr * 64 + (p - y * (uint32_t)g.W)]);
}

// One workgroup of kSelThreads: brackets for the ranks sel.k[0..sel.n), from
// the samples in cand.buf.
template <bool F32>
__device__ __forceinline__ void pct_bracket_wg(uint32_t n, const PctSel &sel, const uint32_t *ranks, void *states,
                                               const Cand &cand) {
    constexpr int PER = kSample / kSelThreads, NT = 2 * kMaxPctSel;
    constexpr int S1 = F32 ? 21 : 5, S2 = F32 ? 10 : 0;  // digits: 11, 11, 10 bits (uint16: 11, 5)
    __shared__ uint32_t h[NT][2048];
    __shared__ uint32_t tkey[NT], trank[NT], tless[NT], teq[NT];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t sn = samples_of(n);
    const bool direct = n <= kDirectPixels;
    const int nt = 2 * sel.n;
    uint32_t key[PER];
    if (!direct) {
#pragma unroll
        for (int j = 0; j < PER; j++) {
            const uint32_t i = (uint32_t)(tid + j * kSelThreads);
            key[j] = glb(cand.buf)[i < sn ? i : 0];
        }
        for (int i = tid; i < 2048; i += kSelThreads) h[0][i] = 0;
        if (tid < nt) {
            int lo, hi;
            sample_ranks(ranks[tid >> 1], n, sn, lo, hi);
            trank[tid] = (uint32_t)min(max(tid & 1 ? hi : lo, 0), (int)sn - 1);
        }
        __syncthreads();
        // first digit: one histogram for all targets
#pragma unroll
        for (int j = 0; j < PER; j++)
            if ((uint32_t)(tid + j * kSelThreads) < sn) hist_add(h[0], key[j] >> S1);
        __syncthreads();
        if (wave < nt) {
            uint32_t r = trank[wave];
            const int b = wave_find(h[0], r);
            if (lane == 0) {
                tkey[wave] = (uint32_t)b << S1;
                tless[wave] = trank[wave] - r;  // keys in lower buckets
                trank[wave] = r;
            }
        }
        // further digits: a histogram per target
#pragma unroll
        for (int level = 1; level < (F32 ? 3 : 2); level++) {
            const int sh = level == 1 ? S2 : 0, above = level == 1 ? S1 : S2;
            const uint32_t dm = (1u << (above - sh)) - 1u;
            __syncthreads();
            for (int i = tid; i < nt * 2048; i += kSelThreads) (&h[0][0])[i] = 0;
            __syncthreads();
            for (int q = 0; q < nt; q++) {
                const uint32_t pre = tkey[q] >> above;
#pragma unroll
                for (int j = 0; j < PER; j++)
                    if ((uint32_t)(tid + j * kSelThreads) < sn && (key[j] >> above) == pre)
                        hist_add(h[q], (key[j] >> sh) & dm);
            }
            __syncthreads();
            if (wave < nt) {
                uint32_t r = trank[wave];
                const int b = wave_find(h[wave], r);
                if (lane == 0) {
                    tkey[wave] |= (uint32_t)b << sh;
                    tless[wave] += trank[wave] - r;
                    trank[wave] = r;
                    teq[wave] = h[wave][b];
                }
            }
        }
        __syncthreads();
    }
    if (tid < sel.n) {
        const int a = 2 * tid, b = a + 1;
        VLG_GLOBAL PctQ *st = qstate(states, sel.slot[tid]);
        uint32_t mode = PCT_DIRECT, lo = 0, hi = 0, ties = 0;
        if (!direct) {
            mode = PCT_LIGHT;
            ties = max(teq[a], teq[b]) >= kTies;
            lo = tkey[a];
            hi = tkey[b];
            int rl, rh;
            sample_ranks(ranks[tid], n, sn, rl, rh);
            // sample keys in the bracket beyond its width: ties
            const uint32_t span = (uint32_t)(min(rh, (int)sn - 1) - max(rl, 0) + 1), in = tless[b] + teq[b] - tless[a];
            // (or more than the candidates' room, a sixteenth, holds with a margin)
            if (in > min(span + span / 2 + 64, sn * 17 / 320)) mode = PCT_HEAVY;
            // ranks near an end: the bracket takes everything on that side
            if (rl < 0) lo = 0;
            if (rh >= (int)sn) hi = kTopKey<F32>;
        }
        st->k = ranks[tid];
        st->lo = lo;
        st->hi = hi;
        st->mode = mode;
        st->nlist = 0;
        st->ties = ties;
    }
    if (!direct)
        for (int q = 0; q < sel.n; q++) {
            VLG_GLOBAL PctQ *st = qstate(states, sel.slot[q]);
            for (int i = tid; i < 2048; i += kSelThreads) st->hist[i] = 0;
            for (int i = tid; i < kList; i += kSelThreads) st->list[i] = 0;
            if (tid < kSegs * 8) (&st->seg[tid >> 3].ncand)[tid & 7] = 0;
        }
    __syncthreads();  // the next image of a persistent workgroup reuses the LDS
}

// The pass over elements [i0, i1) (chunks of 1024) for M ranks.  Per 64
// elements and rank: one subtraction and two compares; the lanes whose key is
// inside append it to the wave's queue in LDS, which goes to the rank's
// candidates in global memory when it is nearly full.  Bound by instruction
// issue (about 15 vector and 20 scalar instructions per 64 elements with
// three ranks) next to the read of the channel.
constexpr int kQueue = 512;  // flushed when four more elements of every lane might not fit
struct WaveSums {  // per wave of a workgroup
    uint32_t cnt[kThreads / 64][kMaxPctSel], below[kThreads / 64][kMaxPctSel], eqlo[kThreads / 64][kMaxPctSel],
        eqhi[kThreads / 64][kMaxPctSel];
    // the places of its candidates: from at[0] on (pieces = 0), or pieces of
    // the rank's segments, piece p from at[p] on for the workgroup's candidates
    // first[p] .. first[p + 1] - 1
    int pieces[kMaxPctSel];
    uint32_t first[kMaxPctSel][kSegs + 1], at[kMaxPctSel][kSegs];
};
template <typename T, int M, bool HEAVY, bool NT, int NSEG>
__device__ __forceinline__ void pct_collect(const Geo &g, const T *img, const PctSel &sel, void *states,
                                            const Cand &cand_, int seg, int64_t i0, int64_t i1,
                                            uint32_t (*queue)[kQueue], WaveSums &sums) {
    const Cand cand{cand_.buf, cand_.cap, NSEG};
    using V = typename Vec4<T>::type;
    constexpr int U = 4;
    constexpr int64_t stride = kThreads * 4;
    const int64_t pitch = (int64_t)g.wpr * 64;
    const int lane = lane_id();
    // keys in [base, base + width] are candidates; HEAVY: the keys next to
    // that range on either side are lo and hi (`below` then counts lo too)
    uint32_t base[M], width[M], cnt[M];
    uint32_t below[M], eqlo[M], eqhi[M];  // of this lane
    uint32_t inner = 0, heavy = 0;  // bit per rank
    int flushes = 0;                // of this wave
#pragma unroll
    for (int j = 0; j < M; j++) {
        const VLG_GLOBAL PctQ *st = qstate(states, sel.slot[j]);
        const uint32_t mode = __builtin_amdgcn_readfirstlane(st->mode);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(st->lo), hi = __builtin_amdgcn_readfirstlane(st->hi);
        const bool hv = mode == PCT_HEAVY;
        if (hv) heavy |= 1u << j;
        if (mode == PCT_LIGHT || (hv && hi - lo >= 2)) inner |= 1u << j;
        base[j] = hv ? lo + 1 : lo;
        width[j] = hv ? hi - lo - 2 : hi - lo;
        below[j] = eqlo[j] = eqhi[j] = cnt[j] = 0;
    }
    auto flush = [&](int j) {
        wave_lds_handoff();
        VLG_GLOBAL PctQ *st = qstate(states, sel.slot[j]);
        // (the flushes of a wave go round the segments)
        const int s = (seg + flushes++) & (NSEG - 1);
        uint32_t at = 0, room = 0;
        if (lane == 0) room = cand.reserve(st, s, cnt[j], at);
        at = __builtin_amdgcn_readfirstlane(at);
        room = __builtin_amdgcn_readfirstlane(room);
        VLG_GLOBAL uint32_t *buf = cand.rank(j) + (size_t)s * cand.seg_cap() + at;
        for (uint32_t i = lane; i < room; i += 64) buf[i] = queue[j][i];
        if (NSEG > 1 && room < cnt[j] && lane == 0)
            __hip_atomic_fetch_add(&st->seg[s].lost, cnt[j] - room, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        cnt[j] = 0;
        wave_lds_handoff();
    };
    for (int64_t c = i0; c < i1; c += U * stride) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = c + u * stride + threadIdx.x * 4;
            v[u] = ld_hint<NT>((const VLG_GLOBAL V *)(glb(img) + (i < i1 ? i : i0)));
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            uint32_t key[4] = {key_of<T>(v[u].x), key_of<T>(v[u].y), key_of<T>(v[u].z), key_of<T>(v[u].w)};
            // elements outside the image count as the largest key (a wave whose
            // 256 elements lie inside one row has none)
            const int64_t iw = c + u * stride + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 256;
            const uint32_t rw = fdiv((uint32_t)(iw >> 6), g.wpr_mul, g.wpr_shift);
            if (iw + 256 > i1 || (int)(iw - (int64_t)rw * pitch) + 256 > g.W) {
                const int64_t i = c + u * stride + threadIdx.x * 4;
                const uint32_t row = fdiv((uint32_t)(i >> 6), g.wpr_mul, g.wpr_shift);
                const int left = i < i1 ? g.W - (int)(i - (int64_t)row * pitch) : 0;
#pragma unroll
                for (int e = 0; e < 4; e++) key[e] = e < left ? key[e] : ~0u;
            }
#pragma unroll
            for (int e = 0; e < 4; e++) {
#pragma unroll
                for (int j = 0; j < M; j++) {
                    // (the counts of the lanes are summed at the end: a
                    // ballot and its population count would fill the scalar
                    // unit, which issues every fourth cycle)
                    const uint32_t t = key[e] - base[j];
                    below[j] += key[e] < base[j];
                    if (HEAVY && (heavy >> j & 1)) {
                        eqlo[j] += t == ~0u;
                        if (width[j] != ~1u) eqhi[j] += t == width[j] + 1;
                    }
                    if (HEAVY && !(inner >> j & 1)) continue;
                    const uint64_t in = __ballot(t <= width[j]);
                    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)in, cnt[j]));
                    if (t <= width[j]) queue[j][at] = key[e];
                    cnt[j] += (uint32_t)__popcll(in);
                }
            }
#pragma unroll
            for (int j = 0; j < M; j++)
                if (cnt[j] > kQueue - 256) flush(j);
        }
    }
    // the workgroup's counts and last candidates together
    const int wave = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < M; j++) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            below[j] += __shfl_xor(below[j], d);
            if (HEAVY) {
                eqlo[j] += __shfl_xor(eqlo[j], d);
                eqhi[j] += __shfl_xor(eqhi[j], d);
            }
        }
        if (lane == 0) {
            sums.cnt[wave][j] = cnt[j];
            sums.below[wave][j] = below[j];
            sums.eqlo[wave][j] = eqlo[j];
            sums.eqhi[wave][j] = eqhi[j];
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < M) {
        const int j = (int)threadIdx.x;
        VLG_GLOBAL PctQ *q = qstate(states, sel.slot[j]);
        VLG_GLOBAL PctSeg *st = &q->seg[seg];
        uint32_t t[4] = {0, 0, 0, 0};
        for (int w = 0; w < kThreads / 64; w++) {
            t[0] += sums.cnt[w][j];
            t[1] += sums.below[w][j];
            t[2] += sums.eqlo[w][j];
            t[3] += sums.eqhi[w][j];
        }
        auto add = [&](VLG_GLOBAL uint32_t *p, uint32_t x) {
            if (x) __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        // (the place first: the other additions overlap its round trip)
        uint32_t at = 0, done = t[0] ? cand.reserve(q, seg, t[0], at) : 0u;
        add(&st->below, t[1] - t[2]);
        add(&st->eqlo, t[2]);
        add(&st->eqhi, t[3]);
        sums.at[j][0] = (uint32_t)seg * cand.seg_cap() + at;
        int n = 0;
        if (NSEG == 1) {
            // (each wave stores what fits)
        } else if (done < t[0]) {
            sums.first[j][0] = 0;
            sums.first[j][n = 1] = done;
            while (n < NSEG && done < t[0]) {
                const int s = (seg + n) & (NSEG - 1);
                done += cand.reserve(q, s, t[0] - done, at);
                sums.at[j][n] = (uint32_t)s * cand.seg_cap() + at;
                sums.first[j][++n] = done;
            }
            add(&st->lost, t[0] - done);
        }
        sums.pieces[j] = n;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < M; j++) {
        uint32_t w0 = 0;  // this wave's first candidate among the workgroup's
        for (int w = 0; w < wave; w++) w0 += sums.cnt[w][j];
        if (NSEG == 1) {
            const uint32_t at = sums.at[j][0] + w0;
            VLG_GLOBAL uint32_t *buf = cand.rank(j);
            for (uint32_t i = lane; i < cnt[j]; i += 64)
                if (at + i < cand.cap) buf[at + i] = queue[j][i];
            continue;
        }
        const int pieces = __builtin_amdgcn_readfirstlane(sums.pieces[j]);
        if (pieces == 0) {  // all in one
            VLG_GLOBAL uint32_t *buf = cand.rank(j) + sums.at[j][0] + w0;
            for (uint32_t i = lane; i < cnt[j]; i += 64) buf[i] = queue[j][i];
        }
        for (int p = 0; p < pieces; p++) {
            const uint32_t p0 = sums.first[j][p], a = max(p0, w0), b = min(sums.first[j][p + 1], w0 + cnt[j]);
            VLG_GLOBAL uint32_t *buf = cand.rank(j) + sums.at[j][p];
            for (uint32_t i = a + lane; i < b; i += 64) buf[i - p0] = queue[j][i - w0];
        }
    }
    __syncthreads();  // the next unit of a persistent workgroup reuses the LDS
}

template <typename T, int M, bool NT, int NSEG>
__device__ __forceinline__ void pct_collect_range(const Geo &g, const T *img, const PctSel &sel, void *states,
                                                  const Cand &cand, int seg, int64_t i0, int64_t i1,
                                                  uint32_t (*queue)[kQueue], WaveSums &sums) {
    if (i0 >= i1 || pixels_of(g) <= kDirectPixels) return;
    bool heavy = false;
    for (int j = 0; j < M; j++)
        heavy |= __builtin_amdgcn_readfirstlane(qstate(states, sel.slot[j])->mode) == PCT_HEAVY;
    if (heavy) pct_collect<T, M, true, NT, NSEG>(g, img, sel, states, cand, seg, i0, i1, queue, sums);
    else pct_collect<T, M, false, NT, NSEG>(g, img, sel, states, cand, seg, i0, i1, queue, sums);
}

// Where a rank stands after the pass (the same in every thread): a key known
// already, or rank r among keys - base of `bits` bits, those of the candidates
// or (rank not bracketed, or too many candidates) the n of the whole channel.
enum PctOf : uint32_t { PCT_KNOWN = 0, PCT_CANDIDATES, PCT_CHANNEL };
struct PctFound {
    PctOf of;
    uint32_t key, r, base, bits, n;
    bool ties;      // equal values are expected (hist_add)
    uint32_t held;  // keys in the lane's segment
};
template <typename T>
__device__ __forceinline__ PctFound pct_found(const Geo &g, const VLG_GLOBAL PctQ *st, const Cand &cand) {
    // (scalars: what follows from them is the same in every lane; the loads first)
    auto scalar = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    const int lane = lane_id();
    const VLG_GLOBAL PctSeg *seg = &st->seg[lane < cand.nseg ? lane : 0];
    uint32_t c = seg->ncand, bl = seg->below, el = seg->eqlo, eh = seg->eqhi, ls = seg->lost;
    const uint32_t mode = scalar(st->mode), lo = scalar(st->lo), hi = scalar(st->hi), k = scalar(st->k);
    const bool heavy = mode == PCT_HEAVY;
    const uint32_t width = heavy ? hi - lo - 2 : hi - lo;
    const PctFound channel{PCT_CHANNEL, 0, k, 0, 8 * sizeof(T), pixels_of(g), true, 0};
    if (mode == PCT_DIRECT) return channel;
    PctFound f{PCT_KNOWN, lo, 0, heavy ? lo + 1 : lo, 0, 0, scalar(st->ties) != 0, 0};
    // sums over the segments
    if (lane >= cand.nseg) c = bl = el = eh = ls = 0;
    f.held = min(c, cand.seg_cap());
    const bool lost = cand.nseg > 1 ? ls != 0 : c > f.held;
    if (cand.nseg > 1) c = f.held + ls;
    const bool over = __any(lost);
#pragma unroll
    for (int d = 1; d < kSegs; d <<= 1) {
        c += __shfl_xor(c, d);
        bl += __shfl_xor(bl, d);
        el += __shfl_xor(el, d);
        eh += __shfl_xor(eh, d);
    }
    f.n = scalar(c);
    const uint32_t below = scalar(bl), eqlo = scalar(el), eqhi = scalar(eh);
    f.bits = width ? 32 - __builtin_clz(width) : 0;
    if (k < below) return channel;
    f.r = k - below;
    if (heavy) {
        if (f.r < eqlo) return f;
        f.r -= eqlo;
    }
    if (f.r < f.n) {
        f.of = PCT_CANDIDATES;
        return over ? channel : f;
    }
    f.r -= f.n;
    f.key = hi;
    return heavy && f.r < eqhi ? f : channel;
}

// This thread's values (keys - f.base) of part `part` of `parts` (for
// candidates a multiple of the segments: slices of one segment each); part < 0:
// all of them.
template <typename T, typename Fn>
__device__ __forceinline__ void each_value(const PctFound &f, const Geo &g, const T *img_, const Cand &cand, int j,
                                           int part, int parts, Fn fn) {
    const uint32_t nthr = blockDim.x;
    // part `at` of `of` equal parts of n
    auto cut = [](uint32_t n, uint32_t at, uint32_t of) { return (uint32_t)((uint64_t)n * at / of); };
    if (f.of == PCT_CHANNEL) {
        constexpr int U = 4;
        const VLG_GLOBAL T *img = glb(img_);
        const uint32_t W = (uint32_t)g.W;
        const int64_t pitch = (int64_t)g.wpr * 64;
        uint32_t i = 0, end = f.n;
        if (part >= 0) {
            i = cut(f.n, (uint32_t)part, (uint32_t)parts);
            end = cut(f.n, (uint32_t)part + 1, (uint32_t)parts);
        }
        for (i += threadIdx.x; i < end; i += U * nthr) {
            T v[U];
#pragma unroll
            for (int k = 0; k < U; k++) {
                const uint32_t p = min(i + k * nthr, end - 1), y = p / W;
                v[k] = img[(int64_t)y * pitch + (p - y * W)];
            }
#pragma unroll
            for (int k = 0; k < U; k++)
                if (i + k * nthr < end) fn(key_of<T>(v[k]));
        }
        return;
    }
    const uint32_t per = (uint32_t)(parts / cand.nseg), cap = cand.seg_cap();
    for (int s = 0; s < cand.nseg; s++) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)f.held, s);
        uint32_t i = 0, end = n;
        if (part >= 0) {
            if ((uint32_t)part / per != (uint32_t)s) continue;
            i = cut(n, (uint32_t)part % per, per);
            end = cut(n, (uint32_t)part % per + 1, per);
        }
        const VLG_GLOBAL uint32_t *c = cand.rank(j) + (size_t)s * cap;
        i += threadIdx.x;
        for (; i + 7 * nthr < end; i += 8 * nthr) {
            uint32_t v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = c[i + k * nthr];
#pragma unroll
            for (int k = 0; k < 8; k++) fn(v[k] - f.base);
        }
        for (; i < end; i += nthr) fn(c[i] - f.base);
    }
}

// Digits of the values (11 bits, 11 and the rest): their low ends.
__device__ __forceinline__ int digit1(uint32_t bits) { return bits > 11 ? (int)bits - 11 : 0; }
__device__ __forceinline__ int digit2(uint32_t bits) { return bits > 22 ? (int)bits - 22 : 0; }

// Many values to choose from: the histogram of their leading digit, `parts`
// workgroups per rank.
__device__ __forceinline__ bool pct_many(const PctFound &f) {
    return f.of == PCT_CHANNEL ? f.n > kDirectPixels : f.of == PCT_CANDIDATES && f.n > kFewCandidates;
}
template <typename T>
__device__ __forceinline__ void pct_value_hist(const Geo &g, const T *img, VLG_GLOBAL PctQ *st, const Cand &cand, int j,
                                               int part, int parts, uint32_t *h) {
    const PctFound f = pct_found<T>(g, st, cand);
    if (!pct_many(f)) return;
    const int sh = digit1(f.bits);
    for (int i = (int)threadIdx.x; i < 2048; i += (int)blockDim.x) h[i] = 0;
    __syncthreads();
    each_value(f, g, img, cand, j, part, parts, [&](uint32_t v) {
        if (f.of == PCT_CHANNEL) hist_add(h, v >> sh);
        else atomicAdd(&h[v >> sh], 1u);
    });
    __syncthreads();
    for (int i = (int)threadIdx.x; i < 2048; i += (int)blockDim.x)
        if (h[i]) __hip_atomic_fetch_add(&st->hist[i], h[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
}

// The bucket of a histogram of 2048 that holds rank r; r: the rank in it.
__device__ __forceinline__ uint32_t pct_bucket(const VLG_GLOBAL uint32_t *hist, uint32_t &r, uint32_t *h,
                                               uint32_t *found) {
    const int tid = (int)threadIdx.x;
    __syncthreads();
    for (int i = tid; i < 2048; i += kSelThreads) h[i] = hist[i];
    __syncthreads();
    if (tid < 64) {
        uint32_t rr = r;
        const int b = wave_find(h, rr);
        if (tid == 0) {
            found[0] = (uint32_t)b;
            found[1] = rr;
        }
    }
    __syncthreads();
    r = found[1];
    return found[0];
}
// Many values: those in the rank's bucket of the leading digit go to the
// state's list, `parts` workgroups of kSelThreads per rank.  A bucket of more
// than the list holds (ties, or keys that crowd into one 2048th of the
// bracket, as flat regions do) is counted by the next digit instead, and by
// the last one in pct_refine: one workgroup going over a million such
// candidates three times made a formula with two ranks at 4096^2 (flat ellipses)
// take 1.16 ms, which takes 0.35 so; where no bucket is crowded the extra launch
// costs 5 us per step, 17 in a batch of 128 images.  A rank that its bracket
// missed is found in the same launches, over the whole channel.
template <typename T>
__device__ __forceinline__ void pct_list(const Geo &g, const T *img, VLG_GLOBAL PctQ *st, const Cand &cand, int j,
                                         int part, int parts, uint32_t *h, uint32_t *found) {
    const PctFound f = pct_found<T>(g, st, cand);
    const int sh = digit1(f.bits), sh2 = digit2(f.bits);
    if (!pct_many(f) || sh == 0) return;
    uint32_t r = f.r;
    const uint32_t bucket = pct_bucket(st->hist, r, h, found);
    if (st->hist[bucket] > (uint32_t)kList) {
        __syncthreads();  // every thread has read found
        for (int i = (int)threadIdx.x; i < 2048; i += kSelThreads) h[i] = 0;
        __syncthreads();
        each_value(f, g, img, cand, j, part, parts, [&](uint32_t v) {
            if (v >> sh == bucket) hist_add(h, (v >> sh2) & ((1u << (sh - sh2)) - 1u));
        });
        __syncthreads();
        for (int i = (int)threadIdx.x; i < 2048; i += kSelThreads)
            if (h[i]) __hip_atomic_fetch_add(&st->list[i], h[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (threadIdx.x == 0) st->nlist = kCrowded;
        __syncthreads();  // h and found are rewritten for the next image
        return;
    }
    // collected in LDS first: one addition to the shared count per workgroup
    __syncthreads();  // every thread has read found
    if (threadIdx.x == 0) found[0] = 0;
    __syncthreads();
    each_value(f, g, img, cand, j, part, parts, [&](uint32_t v) {
        if (v >> sh != bucket) return;
        const uint32_t at = atomicAdd(&found[0], 1u);
        if (at < 2048)
            h[at] = v;
        else  // (the bucket holds at most kList in all)
            st->list[__hip_atomic_fetch_add(&st->nlist, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = v;
    });
    __syncthreads();
    const uint32_t n = found[0] < 2048 ? found[0] : 2048;
    if (threadIdx.x == 0 && n)
        found[1] = __hip_atomic_fetch_add(&st->nlist, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kSelThreads) st->list[found[1] + i] = h[i];
    __syncthreads();  // h and found are rewritten for the next image
}

// The last digit of a crowded bucket (float32): counted behind the second.
template <typename T>
__device__ __forceinline__ void pct_refine(const Geo &g, const T *img, VLG_GLOBAL PctQ *st, const Cand &cand, int j,
                                           int part, int parts, uint32_t *h, uint32_t *found) {
    if (st->nlist != kCrowded) return;
    const PctFound f = pct_found<T>(g, st, cand);
    const int sh = digit1(f.bits), sh2 = digit2(f.bits);
    if (!pct_many(f) || sh2 == 0) return;
    uint32_t r = f.r;
    uint32_t top = pct_bucket(st->hist, r, h, found);
    top = top << (sh - sh2) | pct_bucket(st->list, r, h, found);
    __syncthreads();  // every thread has read found
    for (int i = (int)threadIdx.x; i < 2048; i += kSelThreads) h[i] = 0;
    __syncthreads();
    each_value(f, g, img, cand, j, part, parts, [&](uint32_t v) {
        if (v >> sh2 == top) hist_add(h, v & ((1u << sh2) - 1u));
    });
    __syncthreads();
    for (int i = (int)threadIdx.x; i < 2048; i += kSelThreads)
        if (h[i]) __hip_atomic_fetch_add(&st->list[2048 + i], h[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();  // h and found are rewritten for the next image
}

// The rank's value, one workgroup of kSelThreads: from what the launches above
// counted or listed (spread: they ran, and there were many values), among all
// values (few), or an end of the bracket.
template <typename T>
__device__ __forceinline__ void pct_pick_wg(const Geo &g, const T *img, VLG_GLOBAL PctQ *st, const Cand &cand, int j,
                                            bool spread, VLG_GLOBAL float *result, uint32_t *h, uint32_t *found) {
    const int tid = (int)threadIdx.x;
    PctFound f = pct_found<T>(g, st, cand);
    if (f.of == PCT_CHANNEL && f.n <= kDirectPixels && f.n > 0) {
        // no sample: ties when a wave's first pixels are mostly equal
        const uint32_t W = (uint32_t)g.W, i = min((uint32_t)tid * (f.n / kSelThreads + 1), f.n - 1), y = i / W;
        const uint32_t v = key_of<T>(glb(img)[(int64_t)y * g.wpr * 64 + (i - y * W)]);
        f.ties = __builtin_amdgcn_readfirstlane(__syncthreads_or(__popcll(__ballot(v == (uint32_t)__builtin_amdgcn_readfirstlane((int)v))) > 8));
    }
    uint32_t key = f.key;
    // the rank r value of bits-bit values, 11 bits at a time from the top, over
    // what each(fn) calls fn(value) for
    auto radix = [&](uint32_t bits, uint32_t r, auto each) {
        uint32_t pre = 0;
        int sh = (int)bits;
        while (sh > 0) {
            const int ns = sh > 11 ? sh - 11 : 0;
            const uint32_t dm = (1u << (sh - ns)) - 1u, want = sh < 32 ? pre >> sh : 0u;
            __syncthreads();
            for (int i = tid; i < 2048; i += kSelThreads) h[i] = 0;
            __syncthreads();
            // (two loops: the time of one workgroup is also that of fetching its code)
            auto in = [&](uint32_t v) { return (sh < 32 ? v >> sh : 0u) == want; };
            if (f.ties)
                each([&](uint32_t v) {
                    if (in(v)) hist_add(h, (v >> ns) & dm);
                });
            else
                each([&](uint32_t v) {
                    if (in(v)) atomicAdd(&h[(v >> ns) & dm], 1u);
                });
            __syncthreads();
            if (tid < 64) {
                uint32_t rr = r;
                const int b = wave_find(h, rr);
                if (tid == 0) {
                    found[0] = (uint32_t)b;
                    found[1] = rr;
                }
            }
            __syncthreads();
            pre |= (uint32_t)__builtin_amdgcn_readfirstlane((int)found[0]) << ns;
            r = found[1];
            sh = ns;
        }
        return pre;
    };
    if (spread && pct_many(f)) {
        const int sh = digit1(f.bits), sh2 = digit2(f.bits);
        uint32_t r = f.r, v = pct_bucket(st->hist, r, h, found);
        const uint32_t n = st->nlist;
        if (sh > 0 && n == kCrowded) {
            v = v << (sh - sh2) | pct_bucket(st->list, r, h, found);
            if (sizeof(T) == 4 && sh2 > 0) v = v << sh2 | pct_bucket(st->list + 2048, r, h, found);
        } else if (sh > 0) {
            v = (v << sh) + radix(sh, r, [&](auto fn) {
                    for (uint32_t i = tid; i < n; i += kSelThreads) fn(st->list[i] & ((1u << sh) - 1u));
                });
        }
        key = f.base + v;
    } else if (f.of != PCT_KNOWN) {
        key = f.base + radix(f.bits, f.r, [&](auto fn) { each_value(f, g, img, cand, j, -1, 1, fn); });
    }
    if (tid == 0) *result = value_of<T>(key);
    __syncthreads();  // h and found are rewritten for the next image
}

// ---- single image
template <typename T>
__global__ __launch_bounds__(kThreads) void k_pct_gather(Geo g, const T *img, Cand cand) {
    pct_gather(g, img, cand, blockIdx.x * kThreads + threadIdx.x);
}

template <bool F32>
__global__ __launch_bounds__(kSelThreads) void k_pct_bracket(uint32_t n, PctSel sel, void *states, Cand cand) {
    __shared__ uint32_t ranks[kMaxPctSel];
    if ((int)threadIdx.x < sel.n) ranks[threadIdx.x] = sel.k[threadIdx.x];
    __syncthreads();
    pct_bracket_wg<F32>(n, sel, ranks, states, cand);
}

template <typename T, int M, bool NT, int NSEG>
__global__ __launch_bounds__(kThreads) void k_pct_collect(Geo g, const T *img, PctSel sel, void *states, Cand cand) {
    __shared__ uint32_t queue[kThreads / 64][M][kQueue];
    __shared__ WaveSums sums;
    const int64_t n = (int64_t)g.H * g.wpr * 64, chunks = (n + kThreads * 4 - 1) / (kThreads * 4);
    const int64_t per = (chunks + gridDim.x - 1) / gridDim.x * (kThreads * 4);
    const int64_t i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
    const int seg = (int)((blockIdx.x * 0x9E3779B1u) >> 28) & (NSEG - 1);
    pct_collect_range<T, M, NT, NSEG>(g, img, sel, states, cand, seg, i0, i1, queue[threadIdx.x >> 6], sums);
}

// (blockIdx.x: the part, blockIdx.y: the rank)
template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_pct_candidates(Geo g, const T *img, PctSel sel, void *states,
                                                                Cand cand) {
    __shared__ uint32_t h[2048];
    const int j = (int)blockIdx.y;
    pct_value_hist(g, img, qstate(states, sel.slot[j]), cand, j, (int)blockIdx.x, (int)gridDim.x, h);
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_pct_list(Geo g, const T *img, PctSel sel, void *states, Cand cand) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.y;
    pct_list(g, img, qstate(states, sel.slot[j]), cand, j, (int)blockIdx.x, (int)gridDim.x, h, found);
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_pct_refine(Geo g, const T *img, PctSel sel, void *states, Cand cand) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.y;
    pct_refine(g, img, qstate(states, sel.slot[j]), cand, j, (int)blockIdx.x, (int)gridDim.x, h, found);
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void k_pct_pick(Geo g, const T *img, PctSel sel, void *states, Cand cand,
                                                          bool spread, float *results) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.x;
    pct_pick_wg<T>(g, img, qstate(states, sel.slot[j]), cand, j, spread, glb(results) + sel.slot[j], h, found);
}

// ---- batches: states, results and candidates live in each image's workspace
__device__ __forceinline__ Cand bcand(const BImg &d) {
    return Cand{(uint32_t *)(d.ws + d.off_cand), d.cand_cap, 1};
}
template <typename T>
__device__ __forceinline__ const T *bchan(const BImg &d, int chan) {
    return (const T *)(d.img + (int64_t)chan * d.chan_bytes);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void kb_pct_gather(BatchArgs a, int chan) {
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        pct_gather(d.g, bchan<T>(d, chan), bcand(d), blockIdx.y * kThreads + threadIdx.x);
    }
}

template <bool F32>
__global__ __launch_bounds__(kSelThreads) void kb_pct_bracket(BatchArgs a, PctSel sel) {
    __shared__ uint32_t ranks[kMaxPctSel];
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        if ((int)threadIdx.x < sel.n) ranks[threadIdx.x] = glb(d.ranks)[sel.slot[threadIdx.x]];
        __syncthreads();
        pct_bracket_wg<F32>(pixels_of(d.g), sel, ranks, d.ws + d.off_pctst, bcand(d));
    }
}

// (the waves per SIMD that the queues of two and of three ranks leave room for;
// with five for three ranks the pass of a batch takes 193 us, not 185)
template <typename T, int M, bool NT>
__global__ __launch_bounds__(kThreads, M == 2 ? 7 : M == 3 ? 6 : 1) void kb_pct_collect(BatchArgs a, int chan, PctSel sel) {
    __shared__ uint32_t queue[kThreads / 64][M][kQueue];
    __shared__ WaveSums sums;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        const int64_t n = (int64_t)d.g.H * d.g.wpr * 64, i0 = (u_ - a.prefix[ii]) * kPctUnit;
        pct_collect_range<T, M, NT, 1>(d.g, bchan<T>(d, chan), sel, d.ws + d.off_pctst, bcand(d), 0, i0,
                                    min(i0 + kPctUnit, n), queue[threadIdx.x >> 6], sums);
    }
}

// (blockIdx.y: the rank, blockIdx.z: the part)
template <typename T>
__global__ __launch_bounds__(kSelThreads) void kb_pct_candidates(BatchArgs a, int chan, PctSel sel) {
    __shared__ uint32_t h[2048];
    const int j = (int)blockIdx.y;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        pct_value_hist(d.g, bchan<T>(d, chan), qstate(d.ws + d.off_pctst, sel.slot[j]), bcand(d), j, (int)blockIdx.z,
                       (int)gridDim.z, h);
    }
}

template <typename T>
__global__ __launch_bounds__(kSelThreads, 8) void kb_pct_list(BatchArgs a, int chan, PctSel sel) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.y;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        pct_list(d.g, bchan<T>(d, chan), qstate(d.ws + d.off_pctst, sel.slot[j]), bcand(d), j, (int)blockIdx.z,
                 (int)gridDim.z, h, found);
    }
}

template <typename T>
__global__ __launch_bounds__(kSelThreads) void kb_pct_refine(BatchArgs a, int chan, PctSel sel) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.y;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        pct_refine(d.g, bchan<T>(d, chan), qstate(d.ws + d.off_pctst, sel.slot[j]), bcand(d), j, (int)blockIdx.z,
                   (int)gridDim.z, h, found);
    }
}

template <typename T>
__global__ __launch_bounds__(kSelThreads, 8) void kb_pct_pick(BatchArgs a, int chan, PctSel sel) {
    __shared__ uint32_t h[2048], found[2];
    const int j = (int)blockIdx.y;
    VLG_BATCH_LOOP(a) {
        VLG_BATCH_IMG(a)
        pct_pick_wg<T>(d.g, bchan<T>(d, chan), qstate(d.ws + d.off_pctst, sel.slot[j]), bcand(d), j, true,
                       glb((float *)(d.ws + d.off_pct)) + sel.slot[j], h, found);
    }
}

#define VLG_BY_RANKS(n, K)  \
    switch (n) {            \
    case 1: K(1); break;    \
    case 2: K(2); break;    \
    case 3: K(3); break;    \
    default: K(4); break;   \
    }

template <typename T>
hipError_t percentile_sampled(hipStream_t s, const Geo &g, const T *img, const PctSel &sel, void *states,
                              float *results, Cand cand) {
    constexpr bool F32 = sizeof(T) == 4;
    const int64_t n = (int64_t)g.H * g.wpr * 64;
    const uint32_t npix = pixels_of(g);
    const int grid = grid_for(n, kThreads * 4 * 4, 2048);
    cand.nseg = grid >= 1024 ? kSegs : 1;
    if (npix > kDirectPixels) k_pct_gather<T><<<kSample / kThreads, kThreads, 0, s>>>(g, img, cand);
    k_pct_bracket<F32><<<1, kSelThreads, 0, s>>>(npix, sel, states, cand);
    if (npix > kDirectPixels) {
        const bool nt = n * (int64_t)sizeof(T) > kStreamBytes;
#define K(M)                                                                                              \
    if (nt) k_pct_collect<T, M, true, kSegs><<<grid, kThreads, 0, s>>>(g, img, sel, states, cand);        \
    else if (cand.nseg > 1) k_pct_collect<T, M, false, kSegs><<<grid, kThreads, 0, s>>>(g, img, sel, states, cand); \
    else k_pct_collect<T, M, false, 1><<<grid, kThreads, 0, s>>>(g, img, sel, states, cand)
        VLG_BY_RANKS(sel.n, K)
#undef K
    }
    const bool many = npix > kDirectPixels && cand.cap > kFewCandidates;
    if (many) {
        const dim3 parts(cand.nseg > 1 ? 4 * cand.nseg : 8, sel.n);
        k_pct_candidates<T><<<parts, kSelThreads, 0, s>>>(g, img, sel, states, cand);
        k_pct_list<T><<<parts, kSelThreads, 0, s>>>(g, img, sel, states, cand);
        if (F32) k_pct_refine<T><<<parts, kSelThreads, 0, s>>>(g, img, sel, states, cand);
    }
    k_pct_pick<T><<<sel.n, kSelThreads, 0, s>>>(g, img, sel, states, cand, many, results);
    return hipGetLastError();
}

template <typename T>
hipError_t b_percentile_sampled(hipStream_t s, const BatchArgs &one, int64_t total_one, const BatchArgs &hist,
                                int64_t total_hist, int chan, const PctSel &sel) {
    constexpr bool F32 = sizeof(T) == 4;
    const int g1 = persistent_grid(one, total_one), gh = persistent_grid(hist, total_hist);
    kb_pct_gather<T><<<dim3(g1, kSample / kThreads), kThreads, 0, s>>>(one, chan);
    kb_pct_bracket<F32><<<g1, kSelThreads, 0, s>>>(one, sel);
    const bool nt = total_hist * kPctUnit * (int64_t)sizeof(T) > kStreamBytes;
#define K(M)                                                                         \
    if (nt) kb_pct_collect<T, M, true><<<gh, kThreads, 0, s>>>(hist, chan, sel);     \
    else kb_pct_collect<T, M, false><<<gh, kThreads, 0, s>>>(hist, chan, sel)
    VLG_BY_RANKS(sel.n, K)
#undef K
    const dim3 parts(g1, sel.n, 4);
    kb_pct_candidates<T><<<parts, kSelThreads, 0, s>>>(one, chan, sel);
    kb_pct_list<T><<<parts, kSelThreads, 0, s>>>(one, chan, sel);
    if (F32) kb_pct_refine<T><<<parts, kSelThreads, 0, s>>>(one, chan, sel);
    kb_pct_pick<T><<<dim3(g1, sel.n), kSelThreads, 0, s>>>(one, chan, sel);
    return hipGetLastError();
}
#undef VLG_BY_RANKS

// ------------------------------------------------------------------ radix select
// float32 uses digits of 13, 10 and 9 bits in batches (the first pass has a
// single group, so its histogram takes the LDS of all four) and 11, 11 and 10
// bits on single images (whose workgroups read fewer elements, so a wider
// histogram to clear and add costs more than its fewer LDS conflicts save);
// uint8 one digit of 8 bits, uint16 two.

// Selections of a pass whose digits chosen so far agree share one
// histogram: that of the first of them in the step, whose slot is `src`.
// Passes 0 and 2 count into `a`, pass 1 into `b`, so the selection of pass 1
// can clear `a` while others still read `b`.
struct PctState {
    uint32_t prefix, mask, k, src;
    uint32_t a[8192];
    uint32_t b[2048];
};
static_assert(sizeof(PctState) <= kPctStateBytes, "percentile state");

__device__ void pct_init_wg(PctState *st_, uint32_t k, int slot) {
    VLG_GLOBAL PctState *st = glb(st_);
    for (int i = threadIdx.x; i < 8192; i += blockDim.x) st->a[i] = 0;
    for (int i = threadIdx.x; i < 2048; i += blockDim.x) st->b[i] = 0;
    if (threadIdx.x == 0) {
        st->prefix = 0;
        st->mask = 0;
        st->k = k;
        st->src = (uint32_t)slot;
    }
}

// Histogram the channel elements of the chunks [c, c + 1024) for c = i0,
// i0 + stride, ... below i1 (a channel is stored with pitch wpr*64; i0,
// stride and i1 are multiples of 1024 or of the pitch, so four consecutive
// elements share a row), for the n selections st[0..n): selections whose
// digits chosen so far agree share one LDS histogram (in the first pass all
// of them do), which is then added into the state of the group's first
// selection.
// The streaming part of a histogram pass over elements [i0, i1): MG is the
// number of groups the group test has to try (one in every first pass).
template <typename T, int MG, bool NT>
__device__ __forceinline__ void pct_hist_stream(const Geo &g, const T *__restrict__ img, int m, const uint32_t *pre,
                                                const uint32_t *msk, int shift, int bins, int64_t i0, int64_t i1,
                                                int64_t stride, uint32_t (*h)[2048]) {
    const int64_t pitch = (int64_t)g.wpr * 64;
    const uint32_t dmask = (uint32_t)(bins - 1);
    using V = typename Vec4<T>::type;
    constexpr int U = 8;  // chunks per iteration: U vector loads in flight per thread
    for (int64_t c = i0; c < i1; c += U * stride) {
        V v[U];
        int64_t idx[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            idx[u] = c + u * stride + threadIdx.x * 4;
            v[u] = ld_hint<NT>((const VLG_GLOBAL V *)(glb(img) + (idx[u] < i1 ? idx[u] : i0)));
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = idx[u];
            const bool in = i < i1;
            const uint32_t row = fdiv((uint32_t)(i >> 6), g.wpr_mul, g.wpr_shift);
            const int64_t col = i - (int64_t)row * pitch;
            const float f[4] = {(float)v[u].x, (float)v[u].y, (float)v[u].z, (float)v[u].w};
            uint32_t key[4];
#pragma unroll
            for (int e = 0; e < 4; e++) key[e] = sizeof(T) < 4 ? (uint32_t)f[e] : f32_key(f[e]);
            // the groups of a pass share the digit mask and differ in prefix,
            // so an element belongs to at most one of them
            uint32_t bin[4];
            bool act[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                int grp = -1;
#pragma unroll
                for (int q = MG - 1; q >= 0; q--)
                    if (q < m && (key[e] & msk[q]) == pre[q]) grp = q;
                act[e] = in && col + e < g.W && grp >= 0;
                bin[e] = (uint32_t)max(grp, 0) * 2048u + ((key[e] >> shift) & dmask);
            }
            // four neighbouring elements in one bin (channel values cluster)
            // take one atomic; otherwise each active element adds its own
            uint32_t *hh = &h[0][0];
            if (act[0] && act[1] && act[2] && act[3] && bin[0] == bin[1] && bin[1] == bin[2] && bin[2] == bin[3]) {
                atomicAdd(&hh[bin[0]], 4u);
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    if (act[e]) atomicAdd(&hh[bin[e]], 1u);
            }
        }
    }
}

template <typename T, bool NT>
__device__ void pct_hist_range(const Geo &g, const T *__restrict__ img, PctState *const *st, const int32_t *slot,
                               int n, int pass, int shift, int bins, int64_t i0, int64_t i1, int64_t stride,
                               uint32_t (*h)[2048]) {
    __shared__ uint32_t gpre[kMaxPctSel], gmask[kMaxPctSel];
    __shared__ int rep[kMaxPctSel], first[kMaxPctSel], ngroups;
    if (threadIdx.x == 0) {
        int m = 0;
        for (int j = 0; j < n; j++) {
            const uint32_t p = glb(st[j])->prefix, mk = glb(st[j])->mask;
            int r = -1;
            for (int q = 0; q < m; q++)
                if (gpre[q] == p && gmask[q] == mk) r = q;
            if (r < 0) {
                gpre[m] = p;
                gmask[m] = mk;
                first[m] = j;
                r = m++;
            }
            rep[j] = r;
        }
        ngroups = m;
        // (every workgroup writes the same values)
        for (int j = 0; j < n; j++) glb(st[j])->src = (uint32_t)slot[first[rep[j]]];
    }
    __syncthreads();
    // the group table in registers: the histogram atomics below write LDS, so
    // values left in LDS would be reloaded after every one of them
    const int m = ngroups;
    uint32_t pre[kMaxPctSel], msk[kMaxPctSel];
#pragma unroll
    for (int q = 0; q < kMaxPctSel; q++) {
        pre[q] = q < m ? gpre[q] : 0u;
        msk[q] = q < m ? gmask[q] : 0u;
    }
    // group q's bins at q * 2048 (a single group may take all 8192)
    uint32_t *hh = &h[0][0];
    for (int i = threadIdx.x; i < (m - 1) * 2048 + bins; i += kThreads) hh[i] = 0;
    __syncthreads();
    if (m == 1)
        pct_hist_stream<T, 1, NT>(g, img, m, pre, msk, shift, bins, i0, i1, stride, h);
    else
        pct_hist_stream<T, kMaxPctSel, NT>(g, img, m, pre, msk, shift, bins, i0, i1, stride, h);
    __syncthreads();
    // each group's histogram into its first selection's state
    for (int q = 0; q < m; q++) {
        VLG_GLOBAL uint32_t *gh = pass == 1 ? glb(st[first[q]])->b : glb(st[first[q]])->a;
        for (int i = threadIdx.x; i < bins; i += kThreads) {
            const uint32_t cnt = hh[q * 2048 + i];
            if (cnt) __hip_atomic_fetch_add(&gh[i], cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
}

// one workgroup of 256 threads: find the bucket holding rank k
// (src: the state whose histogram the selection shares in this pass)
__device__ void pct_select_wg(PctState *st_, const PctState *src, int pass, int shift, int bins, int last,
                              int is_int, float *result_, uint32_t *part) {
    VLG_GLOBAL PctState *st = glb(st_);
    VLG_GLOBAL float *result = glb(result_);
    const VLG_GLOBAL uint32_t *hist = pass == 1 ? glb(src)->b : glb(src)->a;
    const int per = bins / kThreads;
    uint32_t local = 0;
    for (int j = 0; j < per; j++) local += hist[threadIdx.x * per + j];
    part[threadIdx.x] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0, k = st->k;
        int t = 0;
        while (t < kThreads - 1 && acc + part[t] <= k) acc += part[t++];
        int b = t * per;
        while (b < t * per + per - 1 && acc + hist[b] <= k) acc += hist[b++];
        st->k = k - acc;
        st->prefix |= (uint32_t)b << shift;
        st->mask |= (uint32_t)(bins - 1) << shift;
        if (last) *result = is_int ? (float)st->prefix : key_f32(st->prefix);
    }
    // `a` is read only by the selections of passes 0 and 2: after pass 1 it
    // is cleared for pass 2
    if (pass == 1)
        for (int i = threadIdx.x; i < 8192; i += kThreads) st->a[i] = 0;
    __syncthreads();
}

__device__ __forceinline__ PctState *sstate(void *states, int slot) {
    return (PctState *)((char *)states + (size_t)slot * kPctStateBytes);
}

__global__ void k_pct_init(PctSel sel, void *states) {
    pct_init_wg(sstate(states, sel.slot[blockIdx.x]), sel.k[blockIdx.x], sel.slot[blockIdx.x]);
}

template <typename T, bool NT>
__global__ __launch_bounds__(kThreads) void k_pct_hist(Geo g, const T *__restrict__ img, PctSel sel, void *states,
                                                       int pass, int shift, int bins) {
    __shared__ uint32_t h[kMaxPctSel][2048];
    PctState *st[kMaxPctSel];
    for (int j = 0; j < sel.n; j++) st[j] = sstate(states, sel.slot[j]);
    // one contiguous range of whole chunks per workgroup: neighbouring
    // pixels share bins, so the histogram a workgroup adds into the state has
    // fewer nonzero bins than that of a strided range
    const int64_t n = (int64_t)g.H * g.wpr * 64, chunks = (n + kThreads * 4 - 1) / (kThreads * 4);
    const int64_t per = (chunks + gridDim.x - 1) / gridDim.x * (kThreads * 4);
    const int64_t i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
    pct_hist_range<T, NT>(g, img, st, sel.slot, sel.n, pass, shift, bins, i0, i1, kThreads * 4, h);
}

__global__ __launch_bounds__(kThreads) void k_pct_select(PctSel sel, void *states, int pass, int shift, int bins,
                                                         int last, int is_int, float *results) {
    __shared__ uint32_t part[kThreads];
    const int slot = sel.slot[blockIdx.x];
    PctState *st = sstate(states, slot);
    pct_select_wg(st, sstate(states, (int)glb(st)->src), pass, shift, bins, last, is_int, results + slot, part);
}

// batch variants: state and result of percentile slot p live in each image's workspace
__device__ __forceinline__ PctState *bstate(const BImg &d, int p) {
    return (PctState *)(d.ws + d.off_pctst + (uint64_t)p * kPctStateBytes);
}

__global__ void kb_pct_init(BatchArgs a, PctSel sel) {
    UnitRange ur(a.prefix, a.n);
    for (int64_t u = ur.begin; u < ur.end; u++) {
        const int ii = ur.img(u);
        for (int j = 0; j < sel.n; j++) {
            pct_init_wg(bstate(a.imgs[ii], sel.slot[j]), a.imgs[ii].ranks[sel.slot[j]], sel.slot[j]);
            __syncthreads();
        }
    }
}

template <typename T, bool NT>
__global__ __launch_bounds__(kThreads) void kb_pct_hist(BatchArgs a, int chan, PctSel sel, int pass, int shift,
                                                        int bins) {
    __shared__ uint32_t h[kMaxPctSel][2048];
    UnitRange ur(a.prefix, a.n);
    for (int64_t u = ur.begin; u < ur.end; u++) {
        const int ii = ur.img(u);
        const BImg d = a.imgs[ii];  // by value (see UnitRange)
        PctState *st[kMaxPctSel];
        for (int j = 0; j < sel.n; j++) st[j] = bstate(d, sel.slot[j]);
        const int64_t i0 = (u - a.prefix[ii]) * kPctUnit;
        const int64_t n = (int64_t)d.g.H * d.g.wpr * 64;
        const int64_t i1 = i0 + kPctUnit < n ? i0 + kPctUnit : n;
        pct_hist_range<T, NT>(d.g, (const T *)(d.img + (int64_t)chan * d.chan_bytes), st, sel.slot, sel.n, pass, shift,
                              bins, i0, i1,
                       kThreads * 4, h);
    }
}

__global__ __launch_bounds__(kThreads) void kb_pct_select(BatchArgs a, PctSel sel, int pass, int shift, int bins,
                                                          int last, int is_int) {
    __shared__ uint32_t part[kThreads];
    const int slot = sel.slot[blockIdx.y];
    UnitRange ur(a.prefix, a.n);
    for (int64_t u = ur.begin; u < ur.end; u++) {
        const int ii = ur.img(u);
        const BImg d = a.imgs[ii];  // by value (see UnitRange)
        PctState *st = bstate(d, slot);
        pct_select_wg(st, bstate(d, (int)glb(st)->src), pass, shift, bins, last, is_int,
                      (float *)(d.ws + d.off_pct) + slot, part);
    }
}

}  // namespace

hipError_t launch_percentile(hipStream_t s, const Geo &g, const void *chan, int dtype, const PctSel &sel,
                             void *states, float *results, uint32_t *cand, uint32_t cap) {
    if (sel.n < 1 || sel.n > kMaxPctSel) return hipErrorInvalidValue;
    // Four ranks of a large uint16 channel keep the radix select: its two passes
    // serve four ranks as fast as one, the sampled pass does not.  us, radix and
    // sampled, a formula with four ranks at 2048^2: 107 / 96 (middle ranks) and
    // 111 / 99 (two of them near the ends); at 3000 x 3100: 131 / 136, 135 / 147;
    // at 5000 x 5100: 158 / 163, 162 / 179; three ranks there: 156 / 141.
    const bool radix = dtype == 2 && sel.n == 4 && (int64_t)g.H * g.W > (1 << 22);
    if (dtype != 1 && g.nwords > 0 && cap > 0 && !radix) {
        const Cand c{cand, cap, 1};
        return dtype == 2 ? percentile_sampled(s, g, (const uint16_t *)chan, sel, states, results, c)
                          : percentile_sampled(s, g, (const float *)chan, sel, states, results, c);
    }
    k_pct_init<<<sel.n, kThreads, 0, s>>>(sel, states);
    const int64_t n = (int64_t)g.H * g.wpr * 64;
    if (n == 0) return hipGetLastError();
    // at least 32 chunks of 1024 elements per workgroup, so that clearing and
    // adding its histogram (up to 8192 bins) stays small next to its reads
    const int grid = grid_for(n, kThreads * 4 * 32, 2048);
    if (dtype == 1) {
        if (n > kStreamBytes) k_pct_hist<uint8_t, true><<<grid, kThreads, 0, s>>>(g, (const uint8_t *)chan, sel, states, 0, 0, 256);
        else k_pct_hist<uint8_t, false><<<grid, kThreads, 0, s>>>(g, (const uint8_t *)chan, sel, states, 0, 0, 256);
        k_pct_select<<<sel.n, kThreads, 0, s>>>(sel, states, 0, 0, 256, 1, 1, results);
        return hipGetLastError();
    }
    if (dtype == 2) {  // uint16: two 8-bit digits
        for (int p = 0; p < 2; p++) {
            if (2 * n > kStreamBytes)
                k_pct_hist<uint16_t, true><<<grid, kThreads, 0, s>>>(g, (const uint16_t *)chan, sel, states, p, 8 - 8 * p, 256);
            else
                k_pct_hist<uint16_t, false><<<grid, kThreads, 0, s>>>(g, (const uint16_t *)chan, sel, states, p, 8 - 8 * p, 256);
            k_pct_select<<<sel.n, kThreads, 0, s>>>(sel, states, p, 8 - 8 * p, 256, p == 1, 1, results);
        }
        return hipGetLastError();
    }
    const int shifts[3] = {21, 10, 0}, bins[3] = {2048, 2048, 1024};
    for (int p = 0; p < 3; p++) {
        if (4 * n > kStreamBytes)
            k_pct_hist<float, true><<<grid, kThreads, 0, s>>>(g, (const float *)chan, sel, states, p, shifts[p], bins[p]);
        else
            k_pct_hist<float, false><<<grid, kThreads, 0, s>>>(g, (const float *)chan, sel, states, p, shifts[p], bins[p]);
        k_pct_select<<<sel.n, kThreads, 0, s>>>(sel, states, p, shifts[p], bins[p], p == 2, 0, results);
    }
    return hipGetLastError();
}

hipError_t launch_b_percentile(hipStream_t s, const BatchArgs &one, int64_t total_one, const BatchArgs &hist,
                               int64_t total_hist, int chan, const PctSel &sel, bool sampled) {
    if (total_one == 0) return hipSuccess;
    if (sel.n < 1 || sel.n > kMaxPctSel) return hipErrorInvalidValue;
    if (sampled && hist.dtype != 1)
        return hist.dtype == 2 ? b_percentile_sampled<uint16_t>(s, one, total_one, hist, total_hist, chan, sel)
                               : b_percentile_sampled<float>(s, one, total_one, hist, total_hist, chan, sel);
    const int g1 = persistent_grid(one, total_one), gh = persistent_grid(hist, total_hist);
    kb_pct_init<<<g1, kThreads, 0, s>>>(one, sel);
    dim3 gs(g1, sel.n);
    // a histogram unit is kPctUnit channel elements
    const bool nt = total_hist * kPctUnit * (hist.dtype == 1 ? 1 : hist.dtype == 2 ? 2 : 4) > kStreamBytes;
    if (hist.dtype == 1) {
        if (nt) kb_pct_hist<uint8_t, true><<<gh, kThreads, 0, s>>>(hist, chan, sel, 0, 0, 256);
        else kb_pct_hist<uint8_t, false><<<gh, kThreads, 0, s>>>(hist, chan, sel, 0, 0, 256);
        kb_pct_select<<<gs, kThreads, 0, s>>>(one, sel, 0, 0, 256, 1, 1);
        return hipGetLastError();
    }
    if (hist.dtype == 2) {  // uint16: two 8-bit digits
        for (int p = 0; p < 2; p++) {
            if (nt) kb_pct_hist<uint16_t, true><<<gh, kThreads, 0, s>>>(hist, chan, sel, p, 8 - 8 * p, 256);
            else kb_pct_hist<uint16_t, false><<<gh, kThreads, 0, s>>>(hist, chan, sel, p, 8 - 8 * p, 256);
            kb_pct_select<<<gs, kThreads, 0, s>>>(one, sel, p, 8 - 8 * p, 256, p == 1, 1);
        }
        return hipGetLastError();
    }
    const int shifts[3] = {19, 9, 0}, bins[3] = {8192, 1024, 512};
    for (int p = 0; p < 3; p++) {
        if (nt) kb_pct_hist<float, true><<<gh, kThreads, 0, s>>>(hist, chan, sel, p, shifts[p], bins[p]);
        else kb_pct_hist<float, false><<<gh, kThreads, 0, s>>>(hist, chan, sel, p, shifts[p], bins[p]);
        kb_pct_select<<<gs, kThreads, 0, s>>>(one, sel, p, shifts[p], bins[p], p == 2, 0);
    }
    return hipGetLastError();
}

}  // namespace vlg
