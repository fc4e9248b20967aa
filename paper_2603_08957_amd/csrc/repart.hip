// Repartition of a tensor relation between two decompositions (Sec. 6: when
// the decomposition an EinSum produces differs from the one its consumer
// reads, the relation is decomposed on all labels promoted in either
// decomposition -- ALLINTS -- and re-composed with the STACK aggregate
// grouped by the consumer's promoted labels).
//
// On the device the two steps are fused: every source tile meets a small box
// of target tiles; the (target key, source tuple) pairs are listed, sorted by
// target key (stable LSD radix sort, so the target keys come out sorted and
// a target's sources in source order; skipped when the listing is already
// in target order, as when row blocks are stacked), run-length encoded into
// the target key set, and each pair copies the intersection of its source
// tile and its target tile (see k_rp_copy).  Target elements no source tile
// covers are zero.
//
// That lists and sorts what a relation with most of its tuples present does
// not need sorted: where both key spaces are of the order of the pairs (see
// cells_ok) the targets are marked in a table over their key space and the
// copy runs over the cells of each target tile -- the source blocks that meet
// it, present or not -- with the source found by its key and absent cells
// written as zeros.  One wait instead of two, no pair list, no zero fill.
// Column panels of 16384 x 32 fp32 as 128 x 128 tiles, 90% of them there
// (1.02 GB moved): the call 535 -> 236 us, of it the copy 229 + 68 us of zero
// fill -> 202 us (5.0 TB/s, about what a large copy reaches); stacking in
// place the 1,048,576 rows between a chain's two EinSums: the chain 2392 -> 2263 us.
#include "tre_internal.h"

#include <algorithm>
#include <cstring>

namespace tre {

namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t n) { return unsigned((n + kThreads - 1) / kThreads); }

constexpr int kRpMaxLabels = kMaxDims;  // labels of one tensor (kept in registers)

// Both decompositions of one tensor, per label position in the label string.
struct RpDesc {
    int32_t nl, rin, rout;
    int32_t pin[kRpMaxLabels], pout[kRpMaxLabels];  // promoted in the source / target
    int64_t ext[kRpMaxLabels], tin[kRpMaxLabels], tout[kRpMaxLabels];
    int64_t sin_[kRpMaxLabels], sout[kRpMaxLabels];  // row-major strides of the source / target tile
    int32_t bits[kRpMaxLabels];                      // bits of each target key attribute (target order)
    int32_t kshift[kRpMaxLabels], kbits[kRpMaxLabels];  // per label: place in the packed target key (0 bits: not promoted)
    int32_t key_bits;
    int64_t te_in, te_out;
    int64_t max_cover;              // target tiles one source tile can meet
    int64_t cover, cells;           // the same, and source tiles one target tile can meet: exact where tiles nest
    int64_t s_in, s_out;            // tuples of a complete source / target relation
    int32_t cmax[kRpMaxLabels];     // cells of a target tile per label
    int32_t regroup;                // a source tile is one contiguous run of its target tile
};

struct RpHeader {
    int32_t err;
    int32_t unsorted;  // nonzero: listing the pairs by source leaves target keys out of order
    int64_t pairs;
    int64_t n_out;
    int32_t multi;  // cells: a source meets more than one target
    int32_t pad0;
    int64_t pad1[4];
};

__device__ inline void source_range(const RpDesc& d, const int32_t* key, int i, int ka, int64_t& lo, int64_t& hi) {
    lo = d.pin[i] ? int64_t(key[ka]) * d.tin[i] : 0;
    hi = lo + d.tin[i];
}

// Packed target key of the target tile holding the lower (upper = false) or
// upper corner of a source tile.
__device__ inline uint64_t corner_key(const RpDesc& d, const int32_t* key, bool upper) {
    uint64_t k = 0;
    int ka = 0, ko = 0;
#pragma unroll
    for (int i = 0; i < kRpMaxLabels; i++) {
        if (i >= d.nl) break;
        int64_t lo, hi;
        source_range(d, key, i, ka, lo, hi);
        ka += d.pin[i];
        if (d.pout[i]) {
            k = (k << d.bits[ko]) | uint64_t((upper ? hi - 1 : lo) / d.tout[i]);
            ko++;
        }
    }
    return k;
}

// Per source tuple: the number of target tiles it meets.  Also flags whether
// listing the pairs source by source (each source's targets in key order)
// already leaves the target keys sorted: it does when no source's first
// target precedes the previous source's last.
__global__ void k_rp_count(const int32_t* __restrict__ keys, int64_t n, RpDesc d, int64_t* __restrict__ cnt,
                           RpHeader* __restrict__ hdr) {
    const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s > n) return;
    if (s == n) {
        cnt[s] = 0;
        return;
    }
    const int32_t* key = keys + s * d.rin;
    int64_t c = 1;
    int ka = 0;
#pragma unroll
    for (int i = 0; i < kRpMaxLabels; i++) {
        if (i >= d.nl) break;
        int64_t lo, hi;
        source_range(d, key, i, ka, lo, hi);
        ka += d.pin[i];
        if (d.pout[i]) c *= (hi - 1) / d.tout[i] - lo / d.tout[i] + 1;
    }
    cnt[s] = c;
    if (s > 0 && corner_key(d, key, false) < corner_key(d, key - d.rin, true)) atomicOr(&hdr->unsorted, 1);
}

// List (target key, source) for every target tile source s meets, in target
// key order within s.
__global__ __launch_bounds__(kThreads) void k_rp_expand(const int32_t* __restrict__ keys, int64_t n, RpDesc d,
                                                        const int64_t* __restrict__ off, uint64_t* __restrict__ tk,
                                                        uint32_t* __restrict__ src) {
    const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int32_t* key = keys + s * d.rin;
    int64_t blo[kRpMaxLabels], bn[kRpMaxLabels];
    int ka = 0;
#pragma unroll
    for (int i = 0; i < kRpMaxLabels; i++) {
        blo[i] = 0;
        bn[i] = 1;
        if (i >= d.nl) continue;
        int64_t lo, hi;
        source_range(d, key, i, ka, lo, hi);
        ka += d.pin[i];
        blo[i] = lo / d.tout[i];
        bn[i] = (hi - 1) / d.tout[i] - blo[i] + 1;
    }
    const int64_t c = off[s + 1] - off[s];
    for (int64_t j = 0; j < c; j++) {
        // digits of j over the target-promoted labels, last label fastest
        int64_t rem = j, block[kRpMaxLabels];
#pragma unroll
        for (int i = kRpMaxLabels - 1; i >= 0; i--) {
            block[i] = blo[i];
            if (i >= d.nl || !d.pout[i]) continue;
            block[i] += rem % bn[i];
            rem /= bn[i];
        }
        uint64_t k = 0;
        int ko = 0;
#pragma unroll
        for (int i = 0; i < kRpMaxLabels; i++) {
            if (i >= d.nl || !d.pout[i]) continue;
            k = (k << d.bits[ko]) | uint64_t(block[i]);
            ko++;
        }
        tk[off[s] + j] = k;
        src[off[s] + j] = uint32_t(s);
    }
}

__global__ void k_rp_heads(const uint64_t* __restrict__ tk, int64_t m, int32_t* __restrict__ flags) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p > m) return;
    flags[p] = (p < m && (p == 0 || tk[p] != tk[p - 1])) ? 1 : 0;
}

__global__ void k_rp_compact(const uint64_t* __restrict__ tk, int64_t m, const int32_t* __restrict__ seg_of,
                             uint64_t* __restrict__ seg_key, RpHeader* hdr) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p > m) return;
    if (p == m) {
        hdr->n_out = seg_of[m];
        return;
    }
    if (p == 0 || tk[p] != tk[p - 1]) seg_key[seg_of[p]] = tk[p];
}

__global__ void k_rp_write_keys(const uint64_t* __restrict__ seg_key, int64_t n_out, RpDesc d,
                                int32_t* __restrict__ keys_out) {
    const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= n_out) return;
    uint64_t k = seg_key[q];
    for (int a = d.rout - 1; a >= 0; a--) {
        keys_out[q * d.rout + a] = int32_t(k & ((uint64_t(1) << d.bits[a]) - 1));
        k >>= d.bits[a];
    }
}

// ------------------------------------------------------------------ cells
// (extents below 2^31 here, so all of it is 32-bit arithmetic)

// One thread per (source tuple, target tile that it may meet): the target's
// mark, and once per source the key checks, its place in the table of source
// keys and the two flags.
__global__ __launch_bounds__(kThreads) void k_rp_mark(const int32_t* __restrict__ keys, int64_t n, RpDesc d,
                                                      int32_t* __restrict__ marks, int32_t* __restrict__ table,
                                                      RpHeader* __restrict__ hdr) {
    const int64_t x = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    const int64_t s = d.cover == 1 ? x : x / d.cover;
    if (s >= n) return;
    uint32_t rem = uint32_t(x - s * d.cover);
    const bool first = rem == 0;
    const int32_t* key = keys + s * d.rin;
    // order against the tuple before (first difference decides)
    int err = 0, order = s > 0 && d.rin > 0 ? 0 : -1;
    uint32_t source = 0, target = 0, low = 0, prev_high = 0, met = 1;
    uint32_t lo_b[kRpMaxLabels], n_b[kRpMaxLabels];
    bool in_range = true;
    int ka = 0;
#pragma unroll
    for (int i = 0; i < kRpMaxLabels; i++) {
        lo_b[i] = 0;
        n_b[i] = 1;
        if (i >= d.nl) continue;
        const uint32_t tin = uint32_t(d.tin[i]), tout = uint32_t(d.tout[i]), gin = uint32_t(d.ext[i] / d.tin[i]);
        int32_t k = 0, kp = 0;
        if (d.pin[i]) {
            k = key[ka];
            if (first && s > 0) {
                kp = key[ka - d.rin];
                if (order == 0 && kp != k) order = kp < k ? -1 : 1;
            }
            in_range = in_range && uint32_t(k) < gin;
            ka++;
        }
        source = source * gin + uint32_t(k);
        if (d.pout[i]) {
            const uint32_t gout = uint32_t(d.ext[i] / d.tout[i]);
            const uint32_t a = uint32_t(k) * tin / tout, b = (uint32_t(k) * tin + tin - 1) / tout;
            lo_b[i] = a;
            n_b[i] = b - a + 1;
            met *= n_b[i];
            low = low * gout + a;
            prev_high = prev_high * gout + (uint32_t(kp) * tin + tin - 1) / tout;
        }
    }
    if (!in_range) err |= 4;
    if (first) {
        if (order == 0) err |= 2;
        if (order > 0) err |= 1;
        if (err) atomicOr(&hdr->err, err);
        if (met > 1) hdr->multi = 1;
        if (s > 0 && low < prev_high) hdr->unsorted = 1;
        if (table && in_range) table[source] = int32_t(s) + 1;
    }
    if (!in_range || rem >= met) return;
    uint32_t place = 1;
#pragma unroll
    for (int i = kRpMaxLabels - 1; i >= 0; i--) {
        if (i >= d.nl || !d.pout[i]) continue;
        uint32_t b = lo_b[i];
        if (n_b[i] > 1) {
            b += rem % n_b[i];
            rem /= n_b[i];
        }
        target += b * place;
        place *= uint32_t(d.ext[i] / d.tout[i]);
    }
    marks[target] = 1;
}

// The marked targets in order, and their number: one workgroup for up to
// 16384 of them, else from the scanned marks.  It has four wavefronts, not
// sixteen: beside another stream's kernel that fills the chip a CU hardly ever
// has sixteen places free at once (the stack of a million-vertex chain's rows
// listed its 4,096 targets only when E1's contraction, 1.4 ms, had ended).
// A wavefront ballots runs of 64 marks, a thread counts one run.
constexpr int kListThreads = 256, kListMax = 64 * kListThreads;
__global__ __launch_bounds__(kListThreads) void k_rp_list_one(const int32_t* __restrict__ marks, int32_t n,
                                                              int32_t* __restrict__ list, RpHeader* __restrict__ hdr) {
    __shared__ int32_t wsum[kListThreads / 64];
    __shared__ uint64_t run[kListThreads];
    __shared__ int32_t at[kListThreads];
    constexpr int kWaves = kListThreads / 64, kBatch = 16;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int runs = ((n + 63) / 64 + kWaves - 1) / kWaves, r0 = w * runs;  // of a wavefront, at most 64
    for (int i0 = 0; i0 < runs; i0 += kBatch) {
        int32_t x[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; i++) x[i] = marks[min((r0 + i0 + i) * 64 + lane, n - 1)];
#pragma unroll
        for (int i = 0; i < kBatch; i++) {
            const uint64_t b = __ballot((r0 + i0 + i) * 64 + lane < n && x[i] != 0);
            if (lane == 0 && i0 + i < runs) run[r0 + i0 + i] = b;
        }
    }
    __syncthreads();
    int32_t total;
    at[threadIdx.x] = block_scan_excl<kListThreads>(int(threadIdx.x) < kWaves * runs ? __popcll(run[threadIdx.x]) : 0, wsum,
                                                    &total);
    __syncthreads();
    const uint64_t below = (uint64_t(1) << lane) - 1;
#pragma unroll 4
    for (int i = 0; i < runs; i++) {
        const uint64_t b = run[r0 + i];
        if (b >> lane & 1) list[at[r0 + i] + __popcll(b & below)] = (r0 + i) * 64 + lane;
    }
    if (threadIdx.x == 0) hdr->n_out = total;
}

__global__ void k_rp_list(const int32_t* __restrict__ off, int64_t n, int32_t* __restrict__ list,
                          RpHeader* __restrict__ hdr) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k == 0) hdr->n_out = off[n];
    if (k < n && off[k + 1] != off[k]) list[off[k]] = int32_t(k);
}

__global__ void k_rp_list_keys(const int32_t* __restrict__ list, int64_t n_out, RpDesc d,
                               int32_t* __restrict__ keys_out) {
    const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= n_out) return;
    uint32_t k = uint32_t(list[q]);
    int ko = d.rout;
#pragma unroll
    for (int i = kRpMaxLabels - 1; i >= 0; i--) {
        if (i >= d.nl || !d.pout[i]) continue;
        const uint32_t g = uint32_t(d.ext[i] / d.tout[i]);
        keys_out[q * d.rout + --ko] = int32_t(k % g);
        k /= g;
    }
}

// The copy: a workgroup takes a run of up to kRpPairs consecutive pairs (or
// cells).  One thread per pair works out the pair's intersection box and cuts
// it into runs that are contiguous in both tiles (the innermost labels, merged
// while the box spans them whole in both tiles); the runs are cut into chunks
// of 16 bytes, or of 4 or one element where a run of the workgroup is shorter.
// A chunk needs no alignment beyond its elements', and the last chunk of a run
// ends where the run ends, so it may copy elements of the chunk before again.
// The chunks of the workgroup's pairs are numbered end to end and the threads
// stride over them with kRpUnroll loads in flight per thread; a chunk's pair
// is found by division when all pairs have the same chunk count, else by
// binary search of the chunk prefix in LDS.
constexpr int kRpPairs = kThreads;
constexpr int kRpUnroll = 4;

struct RpPair {
    int64_t so, to;           // element offset of the box in the source / target tile array
    int32_t run, runs, j;     // elements per contiguous run, runs, first merged label
    int32_t per_run;          // chunks per run
    uint32_t per_run_inv;
    int32_t zero;             // no source: the box is set to zero
    int32_t n[kRpMaxLabels];  // box extent of the unmerged (outer) labels
};

// x / d for x, d < 2^16 by a multiplication: inv = ceil(2^32 / d) (0 for d = 1)
__device__ inline uint32_t div_inv(uint32_t d) { return d > 1 ? 0xffffffffu / d + 1u : 0u; }
__device__ inline int32_t div_by(int32_t x, int32_t d, uint32_t inv, bool small) {
    if (!small) return x / d;
    return inv ? int32_t(__umulhi(uint32_t(x), inv)) : x;
}

template <typename E, int W>
struct RpChunk {
    typedef E type __attribute__((ext_vector_type(W), aligned(sizeof(E))));
};
template <typename E>
struct RpChunk<E, 1> {
    typedef E type;
};

// Copy the chunks [0, total) of the workgroup's pairs, W elements each.
template <typename E, int W>
__device__ inline void rp_copy_chunks(const E* __restrict__ tin, E* __restrict__ tout, const RpDesc& d,
                                      const RpPair* pr, const int32_t* pre, int np, bool uni, int32_t cpp,
                                      int32_t total) {
    using V = typename RpChunk<E, W>::type;
    const bool small = total <= 65536;  // (and so is every divisor)
    const uint32_t cpp_inv = div_inv(uint32_t(cpp));
    for (int32_t c0 = threadIdx.x; c0 < total; c0 += kThreads * kRpUnroll) {
        V v[kRpUnroll];
        int64_t dst[kRpUnroll];
        bool zero[kRpUnroll];
#pragma unroll
        for (int u = 0; u < kRpUnroll; u++) {
            // past the end: copy the last chunk again (the same bytes to the
            // same place), which keeps the loads and stores unconditional
            const int32_t c = min(c0 + u * kThreads, total - 1);
            int i;
            if (uni) {
                i = div_by(c, cpp, cpp_inv, small);
            } else {
                int lo = 0, hi = np;  // pre[lo] <= c < pre[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (pre[mid] <= c) lo = mid;
                    else hi = mid;
                }
                i = lo;
            }
            const RpPair& P = pr[i];
            int32_t x = c - (uni ? i * cpp : pre[i]);
            int64_t os = P.so, ot = P.to;
            if (P.runs > 1) {
                int32_t r = div_by(x, P.per_run, P.per_run_inv, small);
                x -= r * P.per_run;
#pragma unroll
                for (int k = kRpMaxLabels - 2; k >= 0; k--) {
                    if (k >= P.j) continue;
                    int32_t cc = r;
                    if (k > 0) {
                        cc = r % P.n[k];
                        r /= P.n[k];
                    }
                    os += cc * d.sin_[k];
                    ot += cc * d.sout[k];
                }
            }
            const int32_t at = min(x * W, P.run - W);
            zero[u] = P.zero != 0;
            v[u] = *reinterpret_cast<const V*>(tin + os + at);
            dst[u] = ot + at;
        }
#pragma unroll
        for (int u = 0; u < kRpUnroll; u++) *reinterpret_cast<V*>(tout + dst[u]) = zero[u] ? V(0) : v[u];
    }
}

// Where the pairs come from: the sorted list (tk, src, seg_of), or the cells
// of the listed targets.
struct RpWork {
    const int32_t* keys;
    const uint64_t* tk;
    const uint32_t* src;
    const int32_t* seg_of;
    const int32_t* list;   // cells: the targets
    const int32_t* table;  // cells: 1 + source by its key; null: every source is there
    int32_t* keys_out;     // cells
    int64_t m;             // pairs or cells
    int32_t per_wg;
};

template <typename E, bool CELLS>
__global__ __launch_bounds__(kThreads) void k_rp_copy(const E* __restrict__ tin, RpWork wk, RpDesc d,
                                                      E* __restrict__ tout) {
    __shared__ RpPair pr[kRpPairs];
    __shared__ int32_t pre[kRpPairs + 1];
    __shared__ int32_t wsum[kThreads / 64];
    __shared__ int32_t uniform, shortest;
    constexpr int kV = 16 / sizeof(E);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t n_batches = (wk.m + wk.per_wg - 1) / wk.per_wg;
    for (int64_t bt = blockIdx.x; bt < n_batches; bt += gridDim.x) {
        const int64_t p0 = bt * wk.per_wg;
        const int np = int(min<int64_t>(wk.per_wg, wk.m - p0));
        if (tid == 0) {
            uniform = 1;
            shortest = 0x7fffffff;
        }
        __syncthreads();
        if (tid < np) {
            const int64_t p = p0 + tid;
            // intersection box: per label, start in source and target, and length
            int32_t n[kRpMaxLabels];
            int64_t so = 0, to = 0;
            bool zero = false, empty = false;
            if constexpr (CELLS) {
                const int64_t q = p / d.cells;
                uint32_t cell = uint32_t(p - q * d.cells), k = uint32_t(wk.list[q]);
                const bool first = cell == 0;
                int ko = d.rout;
                uint32_t source = 0, place = 1;
#pragma unroll
                for (int i = kRpMaxLabels - 1; i >= 0; i--) {
                    n[i] = 1;
                    if (i >= d.nl) continue;
                    const uint32_t ti = uint32_t(d.tin[i]), tu = uint32_t(d.tout[i]);
                    uint32_t tlo = 0;
                    if (d.pout[i]) {
                        const uint32_t g = uint32_t(d.ext[i] / d.tout[i]), b = k % g;
                        k /= g;
                        tlo = b * tu;
                        ko--;
                        if (first) wk.keys_out[q * d.rout + ko] = int32_t(b);
                    }
                    const uint32_t thi = tlo + tu;
                    uint32_t blk = 0;
                    if (d.pin[i]) {
                        blk = tlo / ti + cell % uint32_t(d.cmax[i]);
                        cell /= uint32_t(d.cmax[i]);
                    }
                    const uint32_t slo = blk * ti, a = max(slo, tlo), e = min(slo + ti, thi);
                    empty = empty || slo >= thi;
                    n[i] = int32_t(e) - int32_t(a);
                    so += int64_t(a - slo) * d.sin_[i];
                    to += int64_t(a - tlo) * d.sout[i];
                    source += blk * place;
                    place *= uint32_t(d.ext[i] / d.tin[i]);
                }
                int64_t s = 0;
                if (!empty) {
                    s = wk.table ? int64_t(wk.table[source]) - 1 : int64_t(source);
                    zero = s < 0;
                }
                // (an absent source: the loads go to the first tile, and are not used)
                so += max<int64_t>(s, 0) * d.te_in;
                to += q * d.te_out;
            } else {
                // the pair's target tuple: segments are numbered by an exclusive
                // scan of the head flags, so pair p belongs to segment seg_of[p + 1] - 1
                const int64_t s = wk.src[p], q = wk.seg_of[p + 1] - 1;
                const int32_t* key = wk.keys + s * d.rin;
                // target block of each target-promoted label, from the packed key
                const uint64_t k = wk.tk[p];
                so = s * d.te_in;
                to = q * d.te_out;
                int ka = 0;
#pragma unroll
                for (int i = 0; i < kRpMaxLabels; i++) {
                    n[i] = 1;
                    if (i >= d.nl) continue;
                    int64_t slo, shi;
                    source_range(d, key, i, ka, slo, shi);
                    ka += d.pin[i];
                    const int64_t block = int64_t((k >> d.kshift[i]) & ((uint64_t(1) << d.kbits[i]) - 1));
                    const int64_t tlo = d.pout[i] ? block * d.tout[i] : 0, thi = tlo + d.tout[i];
                    const int64_t a = max(slo, tlo);
                    n[i] = int32_t(min(shi, thi) - a);
                    so += (a - slo) * d.sin_[i];
                    to += (a - tlo) * d.sout[i];
                }
            }
            // merge labels, innermost first, into one contiguous run while
            // each next label steps exactly one run in both tiles
            int j = d.nl;
            int64_t run = 1;
            bool open = true;
#pragma unroll
            for (int i = kRpMaxLabels - 1; i >= 0; i--) {
                if (i >= d.nl || !open) continue;
                if (j == d.nl || (d.sin_[i] == run && d.sout[i] == run)) {
                    run *= n[i];
                    j = i;
                } else {
                    open = false;
                }
            }
            int32_t runs = 1;
            RpPair& P = pr[tid];
#pragma unroll
            for (int i = 0; i < kRpMaxLabels; i++) {
                P.n[i] = 1;
                if (i >= j) continue;
                P.n[i] = n[i];
                runs *= n[i];
            }
            P.so = so;
            P.to = to;
            P.run = int32_t(run);
            P.runs = empty ? 0 : runs;
            P.j = j;
            P.zero = zero;
            if (!empty && run < kV) atomicMin(&shortest, int32_t(run));
        }
        __syncthreads();
        // chunk counts (all pairs cut alike) and their exclusive scan
        const int32_t width = shortest >= kV ? kV : shortest >= 4 ? 4 : 1;
        int32_t chunks = 0;
        if (tid < np) {
            const int32_t per_run = max((pr[tid].run + width - 1) / width, 1);
            pr[tid].per_run = per_run;
            pr[tid].per_run_inv = div_inv(uint32_t(per_run));
            chunks = pr[tid].runs * per_run;
        }
        int32_t incl = chunks;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        int32_t excl = incl - chunks;
        for (int i = 0; i < w; i++) excl += wsum[i];
        if (tid < np) {
            pre[tid] = excl;
            if (tid == np - 1) pre[np] = excl + chunks;
            if (chunks != pr[0].runs * pr[0].per_run) uniform = 0;
        }
        __syncthreads();
        const int32_t total = pre[np];
        const int32_t cpp = pr[0].runs * pr[0].per_run;
        const bool uni = uniform != 0 && cpp > 0;
        if (width == kV) rp_copy_chunks<E, kV>(tin, tout, d, pr, pre, np, uni, cpp, total);
        else if (width == 4) rp_copy_chunks<E, 4>(tin, tout, d, pr, pre, np, uni, cpp, total);
        else rp_copy_chunks<E, 1>(tin, tout, d, pr, pre, np, uni, cpp, total);
        __syncthreads();  // pr, pre and the flags are rewritten by the next batch
    }
}

// Workgroups of the copy: pairs per workgroup for about kBatchBytes of chunks
// each (a pair averages `pair_bytes`), at most one pair per thread, chunk
// numbers within int32; the grid fills 256 CUs and loops over the rest.  The
// whole call for 16384 x 32 panels to 128 x 128 tiles: 276, 240, 241 and 247 us
// with 16, 32, 64 and 128 KB.
constexpr int64_t kBatchBytes = int64_t(32) << 10;

template <bool CELLS>
hipError_t launch_copy(const RpDesc& d, RpWork wk, int64_t pair_bytes, int32_t elem_bytes, const void* tiles_in,
                       void* tiles_out, hipStream_t s) {
    const int64_t per_wg = std::max<int64_t>(1, kBatchBytes / std::max<int64_t>(1, pair_bytes));
    wk.per_wg = int32_t(std::min<int64_t>(
        {per_wg, kRpPairs, std::max<int64_t>(1, (int64_t(1) << 30) / std::min(d.te_in, d.te_out))}));
    const int64_t batches = (wk.m + wk.per_wg - 1) / wk.per_wg;
    const unsigned grid = unsigned(std::min<int64_t>(batches, 8192));
    if (elem_bytes == 2)
        k_rp_copy<uint16_t, CELLS><<<grid, kThreads, 0, s>>>(reinterpret_cast<const uint16_t*>(tiles_in), wk, d,
                                                              reinterpret_cast<uint16_t*>(tiles_out));
    else
        k_rp_copy<uint32_t, CELLS><<<grid, kThreads, 0, s>>>(reinterpret_cast<const uint32_t*>(tiles_in), wk, d,
                                                              reinterpret_cast<uint32_t*>(tiles_out));
    return hipGetLastError();
}

tre_status dev_fail(hipError_t e, const char* where) {
    set_error(std::string("tre_repartition: ") + where + ": " + hipGetErrorString(e));
    return TRE_E_DEVICE;
}

int32_t bit_width(int64_t x) {
    int32_t b = 0;
    while (x > 0) {
        b++;
        x >>= 1;
    }
    return b;
}

tre_status make_desc(const char* labels, const char* up_in, const char* up_out, const int64_t* extent,
                     const int32_t* tile_in, const int32_t* tile_out, RpDesc& d) {
    std::memset(&d, 0, sizeof(d));
    if (!labels || !up_in || !up_out || !extent || !tile_in || !tile_out) {
        set_error("tre_repartition: null argument");
        return TRE_E_ARG;
    }
    bool seen[26] = {}, in_up[26] = {}, out_up[26] = {};
    int lab[26];
    for (const char* c = labels; *c; c++) {
        if (*c < 'a' || *c > 'z' || seen[*c - 'a']) {
            set_error("tre_repartition: labels must be distinct lower-case letters");
            return TRE_E_PARSE;
        }
        if (d.nl == kRpMaxLabels) {
            set_error("tre_repartition: at most 8 labels");
            return TRE_E_SHAPE;
        }
        seen[*c - 'a'] = true;
        lab[d.nl++] = *c - 'a';
    }
    for (int pass = 0; pass < 2; pass++) {
        for (const char* c = pass ? up_out : up_in; *c; c++) {
            if (*c < 'a' || *c > 'z' || !seen[*c - 'a']) {
                set_error("tre_repartition: a promoted label is not a label of the tensor");
                return TRE_E_SPLIT;
            }
            (pass ? out_up : in_up)[*c - 'a'] = true;
        }
    }
    d.te_in = d.te_out = 1;
    d.max_cover = d.cover = d.cells = d.s_in = d.s_out = 1;
    // blocks of size t met by an aligned run of length len
    auto met = [](int64_t ext, int64_t len, int64_t t) {
        return t % len == 0 ? 1 : len % t == 0 ? len / t : std::min<int64_t>(ext / t, (len - 1) / t + 2);
    };
    auto times = [](int64_t a, int64_t b) { return a > (int64_t(1) << 40) / b ? int64_t(1) << 40 : a * b; };
    for (int i = 0; i < d.nl; i++) {
        const int l = lab[i];
        d.ext[i] = extent[l];
        d.pin[i] = in_up[l];
        d.pout[i] = out_up[l];
        d.tin[i] = in_up[l] ? tile_in[l] : extent[l];
        d.tout[i] = out_up[l] ? tile_out[l] : extent[l];
        if (d.ext[i] < 1 || d.tin[i] < 1 || d.tout[i] < 1 || d.ext[i] % d.tin[i] || d.ext[i] % d.tout[i]) {
            set_error("tre_repartition: every tile size must divide its label's extent");
            return TRE_E_SHAPE;
        }
        d.rin += d.pin[i];
        if (d.pout[i]) {
            d.bits[d.rout] = bit_width(d.ext[i] / d.tout[i] - 1);
            d.key_bits += d.bits[d.rout];
            d.rout++;
            // blocks of size tout met by an aligned run of length tin
            d.max_cover *= std::min<int64_t>(d.ext[i] / d.tout[i], (d.tin[i] - 1) / d.tout[i] + 2);
        }
        if (d.pout[i]) {
            d.cover = times(d.cover, met(d.ext[i], d.tin[i], d.tout[i]));
            d.s_out = times(d.s_out, d.ext[i] / d.tout[i]);
        }
        d.cmax[i] = 1;
        if (d.pin[i]) {
            const int64_t c = met(d.ext[i], d.tout[i], d.tin[i]);
            d.cmax[i] = int32_t(std::min<int64_t>(c, int64_t(1) << 30));
            d.cells = times(d.cells, c);
            d.s_in = times(d.s_in, d.ext[i] / d.tin[i]);
        }
        if (d.tin[i] > (int64_t(1) << 30) / d.te_in || d.tout[i] > (int64_t(1) << 30) / d.te_out) {
            set_error("tre_repartition: a tile holds more than 2^30 elements");
            return TRE_E_SHAPE;
        }
        d.te_in *= d.tin[i];
        d.te_out *= d.tout[i];
    }
    if (d.key_bits > 64) {
        set_error("tre_repartition: target key space exceeds 64 bits");
        return TRE_E_SHAPE;
    }
    // A source tile is one contiguous run of the target tile (row-major) when,
    // at the first label whose source tile is shorter than the target's, every
    // label before it has a source tile of 1 and every label after it the
    // target's tile.  Sources of one target then sit in source key order.
    d.regroup = 1;
    int first = 0;
    while (first < d.nl && d.tin[first] >= d.tout[first]) first++;
    for (int i = 0; i < d.nl; i++)
        if (i < first ? d.tin[i] != 1 : (i > first && d.tin[i] != d.tout[i])) d.regroup = 0;
    if (first == d.nl) {  // no source tile shorter than its target: the same tiles
        d.regroup = 1;
        for (int i = 0; i < d.nl; i++)
            if (d.tin[i] != d.tout[i]) d.regroup = 0;
    }
    int64_t si = 1, so = 1;
    for (int i = d.nl - 1, sh = 0, ko = d.rout - 1; i >= 0; i--) {
        if (d.pout[i]) {
            d.kbits[i] = d.bits[ko--];
            d.kshift[i] = sh;
            sh += d.kbits[i];
        }
        d.sin_[i] = si;
        d.sout[i] = so;
        si *= d.tin[i];
        so *= d.tout[i];
    }
    return TRE_OK;
}

struct RpLayout {
    size_t hdr, cnt, tmp, tk, tk_alt, src, src_alt, hist, seg_of, seg_key, total;
};

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

RpLayout rp_layout(const RpDesc& d, int64_t n_in) {
    const int64_t m = std::max<int64_t>(n_in * d.max_cover, 1);
    RpLayout L{};
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off += align256(std::max<size_t>(b, 1));
        return o;
    };
    L.hdr = take(sizeof(RpHeader));
    L.cnt = take(sizeof(int64_t) * size_t(n_in + 1));
    L.tmp = take(sizeof(int64_t) * scan_tmp_elems(std::max<int64_t>(n_in, m) + 1));
    L.tk = take(sizeof(uint64_t) * size_t(m));
    L.tk_alt = take(sizeof(uint64_t) * size_t(m));
    L.src = take(sizeof(uint32_t) * size_t(m));
    L.src_alt = take(sizeof(uint32_t) * size_t(m));
    L.hist = take(sizeof(int32_t) * size_t(radix_hist_elems(m)));
    L.seg_of = take(sizeof(int32_t) * size_t(m + 1));
    L.seg_key = take(sizeof(uint64_t) * size_t(m));
    L.total = off;
    return L;
}

// Whether the copy runs over the cells of the target tiles: extents and key
// spaces in 32 bits, at least half of the source tuples there (every cell is
// looked at: with fewer, listing the pairs that exist is less work), and the
// marks, the table and the target list within the arrays of the pair list.
bool cells_ok(const RpDesc& d, int64_t n_in) {
    for (int i = 0; i < d.nl; i++)
        if (d.ext[i] > 0x7fffffff) return false;
    const int64_t m = n_in * d.max_cover;
    return d.s_in <= 2 * n_in && d.s_out < 2 * m && d.s_out <= 0x7fffffff &&
           scan_tmp_elems(d.s_out + 1) <= 2 * scan_tmp_elems(std::max<int64_t>(n_in, m) + 1);
}

}  // namespace

}  // namespace tre

using namespace tre;

extern "C" {

size_t tre_repartition_workspace_bytes(const char* labels, const char* upper_in, const char* upper_out,
                                       const int64_t extent[26], const int32_t tile_in[26],
                                       const int32_t tile_out[26], int64_t n_in) {
    RpDesc d;
    if (n_in < 0 || make_desc(labels, upper_in, upper_out, extent, tile_in, tile_out, d) != TRE_OK) return 0;
    return rp_layout(d, n_in).total;
}

tre_status tre_repartition(const char* labels, const char* upper_in, const char* upper_out,
                           const int64_t extent[26], const int32_t tile_in[26], const int32_t tile_out[26],
                           int32_t elem_bytes, const int32_t* keys_in, int64_t n_in, const void* tiles_in,
                           int32_t* keys_out, void* tiles_out, int64_t out_cap, int64_t* n_out, void* ws,
                           size_t ws_bytes, void* stream) {
    RpDesc d;
    tre_status st = make_desc(labels, upper_in, upper_out, extent, tile_in, tile_out, d);
    if (st != TRE_OK) return st;
    if (!n_out || n_in < 0 || out_cap < 0 || (elem_bytes != 2 && elem_bytes != 4)) {
        set_error("tre_repartition: null n_out, negative size or elem_bytes not 2 / 4");
        return TRE_E_ARG;
    }
    *n_out = 0;
    if (n_in == 0) return TRE_OK;
    if (d.rin == 0 && n_in > 1) {
        set_error("tre_repartition: a relation without promoted labels holds at most one tuple");
        return TRE_E_DUPKEY;
    }
    if ((d.rin > 0 && !keys_in) || !tiles_in || !ws || (reinterpret_cast<uintptr_t>(ws) & 255)) {
        set_error("tre_repartition: null keys / tiles / workspace, or workspace not 256-byte aligned");
        return TRE_E_ARG;
    }
    if (n_in * d.max_cover > int64_t(0xffffffffll) || n_in > int64_t(0x7fffffff)) {
        set_error("tre_repartition: too many tuples");
        return TRE_E_SHAPE;
    }
    const RpLayout L = rp_layout(d, n_in);
    if (ws_bytes < L.total) {
        set_error("tre_repartition: workspace too small");
        return TRE_E_WORKSPACE;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* w = reinterpret_cast<char*>(ws);
    RpHeader* hdr = reinterpret_cast<RpHeader*>(w + L.hdr);
    int64_t* cnt = reinterpret_cast<int64_t*>(w + L.cnt);
    uint64_t* tk = reinterpret_cast<uint64_t*>(w + L.tk);
    uint32_t* src = reinterpret_cast<uint32_t*>(w + L.src);
    int32_t* seg_of = reinterpret_cast<int32_t*>(w + L.seg_of);
    uint64_t* seg_key = reinterpret_cast<uint64_t*>(w + L.seg_key);
    hipError_t e;
    RpHeader h{};
    auto bad_keys = [&] {
        set_error("tre_repartition: source keys out of range, unsorted or repeated");
        return (h.err & 4) ? TRE_E_KEYRANGE : (h.err & 1) ? TRE_E_UNSORTED : TRE_E_DUPKEY;
    };
    const bool in_place = tiles_out == tiles_in;
    // the target count is known: whether the caller's buffers take it.  In
    // place, only a regrouping of whole source tiles, in source order, with
    // nothing missing, leaves the bytes where they are (`one`: every source
    // meets one target)
    auto check_out = [&](bool one) {
        *n_out = h.n_out;
        if (in_place && !(d.regroup && !h.unsorted && one && n_in * d.te_in == h.n_out * d.te_out)) {
            set_error("tre_repartition: tiles_out == tiles_in needs every target tile to be its source tiles, "
                      "complete and in source order");
            return TRE_E_ARG;
        }
        if (h.n_out > out_cap) {
            set_error("tre_repartition: output capacity below the target tuple count");
            return TRE_E_CAPACITY;
        }
        if ((d.rout > 0 && !keys_out) || !tiles_out) {
            set_error("tre_repartition: null output buffers");
            return TRE_E_ARG;
        }
        return TRE_OK;
    };
    if (cells_ok(d, n_in)) {
        int32_t* marks = reinterpret_cast<int32_t*>(w + L.tk);
        // (tk_alt follows tk: each holds two words per pair)
        int32_t* table = d.s_in == n_in ? nullptr : marks + d.s_out + 1;
        int32_t* list = reinterpret_cast<int32_t*>(w + L.seg_key);
        const size_t marks_bytes = sizeof(int32_t) * size_t(d.s_out + 1 + (table ? d.s_in : 0));
        if ((e = launch_fill_zero2(hdr, sizeof(RpHeader), marks, marks_bytes, s)) != hipSuccess)
            return dev_fail(e, "header");
        k_rp_mark<<<blocks_for(n_in * d.cover), kThreads, 0, s>>>(keys_in, n_in, d, marks, table, hdr);
        if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "marks");
        if (d.s_out <= kListMax) {
            k_rp_list_one<<<1, kListThreads, 0, s>>>(marks, int32_t(d.s_out), list, hdr);
        } else {
            if ((e = scan_exclusive_i32(marks, marks, d.s_out + 1, reinterpret_cast<int32_t*>(w + L.tmp), s)) !=
                hipSuccess)
                return dev_fail(e, "scan");
            k_rp_list<<<blocks_for(d.s_out), kThreads, 0, s>>>(marks, d.s_out, list, hdr);
        }
        if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "targets");
        if ((e = hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return dev_fail(e, "target count read-back");
        if (h.err) return bad_keys();
        if ((st = check_out(!h.multi)) != TRE_OK) return st;
        if (in_place) {
            if (d.rout > 0) k_rp_list_keys<<<blocks_for(h.n_out), kThreads, 0, s>>>(list, h.n_out, d, keys_out);
            e = hipGetLastError();
        } else {
            RpWork wk{};
            wk.list = list;
            wk.table = table;
            wk.keys_out = keys_out;
            wk.m = h.n_out * d.cells;
            e = launch_copy<true>(d, wk, d.te_out * elem_bytes / d.cells, elem_bytes, tiles_in, tiles_out, s);
        }
        return e == hipSuccess ? TRE_OK : dev_fail(e, "copy");
    }
    // keys: sorted, unique and in range (the relation conventions)
    if ((e = launch_fill_zero(hdr, sizeof(RpHeader), s)) != hipSuccess) return dev_fail(e, "header");
    if (d.rin > 0) {
        int32_t radix[26];
        for (int i = 0, ka = 0; i < d.nl; i++)
            if (d.pin[i]) radix[ka++] = int32_t(d.ext[i] / d.tin[i]);
        if ((e = launch_validate(keys_in, n_in, d.rin, radix, &hdr->err, s)) != hipSuccess)
            return dev_fail(e, "validate");
    }
    k_rp_count<<<blocks_for(n_in + 1), kThreads, 0, s>>>(keys_in, n_in, d, cnt, hdr);
    if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "count");
    if ((e = scan_exclusive_i64(cnt, cnt, n_in + 1, reinterpret_cast<int64_t*>(w + L.tmp), s)) != hipSuccess)
        return dev_fail(e, "scan");
    if ((e = hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(&h.pairs, cnt + n_in, sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return dev_fail(e, "count read-back");
    if (h.err) return bad_keys();
    const int64_t m = h.pairs;
    k_rp_expand<<<blocks_for(n_in), kThreads, 0, s>>>(keys_in, n_in, d, cnt, tk, src);
    if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "expand");
    // the listing is in source order; sort it by target key unless that
    // order already has the target keys sorted (then the stable sort would
    // leave it as it is)
    if (h.unsorted) {
        if ((e = radix_sort_u64(tk, src, reinterpret_cast<uint64_t*>(w + L.tk_alt),
                                reinterpret_cast<uint32_t*>(w + L.src_alt), m, d.key_bits,
                                reinterpret_cast<int32_t*>(w + L.hist), reinterpret_cast<int32_t*>(w + L.tmp), s)) !=
            hipSuccess)
            return dev_fail(e, "sort");
        if (radix_result_in_alt(m, d.key_bits)) {
            tk = reinterpret_cast<uint64_t*>(w + L.tk_alt);
            src = reinterpret_cast<uint32_t*>(w + L.src_alt);
        }
    }
    k_rp_heads<<<blocks_for(m + 1), kThreads, 0, s>>>(tk, m, seg_of);
    if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "heads");
    if ((e = scan_exclusive_i32(seg_of, seg_of, m + 1, reinterpret_cast<int32_t*>(w + L.tmp), s)) != hipSuccess)
        return dev_fail(e, "segments");
    k_rp_compact<<<blocks_for(m + 1), kThreads, 0, s>>>(tk, m, seg_of, seg_key, hdr);
    if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "compact");
    if ((e = hipMemcpyAsync(&h, hdr, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return dev_fail(e, "target count read-back");
    if ((st = check_out(m == n_in)) != TRE_OK) return st;
    if (in_place) {
        if (d.rout > 0) {
            k_rp_write_keys<<<blocks_for(h.n_out), kThreads, 0, s>>>(seg_key, h.n_out, d, keys_out);
            if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "keys");
        }
        return TRE_OK;
    }
    // source tiles are disjoint, so they cover n_in x tile_elems_in target
    // positions; zero the targets only when that leaves some uncovered
    if (n_in * d.te_in < h.n_out * d.te_out &&
        (e = launch_fill_zero(tiles_out, size_t(h.n_out) * size_t(d.te_out) * size_t(elem_bytes), s)) != hipSuccess)
        return dev_fail(e, "zero fill");
    if (d.rout > 0) {
        k_rp_write_keys<<<blocks_for(h.n_out), kThreads, 0, s>>>(seg_key, h.n_out, d, keys_out);
        if ((e = hipGetLastError()) != hipSuccess) return dev_fail(e, "keys");
    }
    RpWork wk{};
    wk.keys = keys_in;
    wk.tk = tk;
    wk.src = src;
    wk.seg_of = seg_of;
    wk.m = m;
    // (the boxes partition the source tiles)
    if ((e = launch_copy<false>(d, wk, n_in * d.te_in * elem_bytes / m, elem_bytes, tiles_in, tiles_out, s)) != hipSuccess)
        return dev_fail(e, "copy");
    return TRE_OK;
}

}  // extern "C"
