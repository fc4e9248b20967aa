// Tile contraction for tiles of any size and label order, bf16 or fp32: the
// GEMM class outside the 128x128 path.  W[b,m,n] += sum_k A[b,m,k] B[b,k,n]
// for every pair of a work unit, on v_mfma_f32_32x32x16_bf16; fp32 operands
// are split into three bf16 parts in registers (split_f32.h), and blocks for
// which that does not hold run again on v_mfma_f32_32x32x2_f32.
//
// One wavefront holds a block of TM x TN MFMA tiles (32 x 32 each).  The
// unit's contraction is cut into chunks of 64 bytes of k (16 fp32, 32 bf16) of
// one pair, and each wavefront copies its own chunks of both operands into a
// private double-buffered stage of LDS (global_load_lds, no registers) and
// reads its fragments from there: no barrier in the main loop.  Reading the
// fragments straight from memory instead -- one row per lane -- was measured:
// every lane's 16 bytes then are an access of their own and the vector L1, at
// one access per cycle, is busy three quarters of the time (335 accesses per
// chunk instead of 128).
//
// Long units: the four wavefronts of a workgroup take every fourth chunk of
// one block and add their sums through LDS in wavefront order; short units:
// every wavefront takes a block of its own (tile_time below).  A chunk that
// would run past K starts at K - 16 (32) instead, with the k that the chunk
// before took set to zero, so all of it is in bounds.
//
// Measured against 64 x 64 blocks staged through registers for a workgroup, on
// the fp32 MFMAs (bf16: two MFMAs a barrier): a chain of 64 x 64 fp32 tiles
// against 100 columns (67 GFLOP, 1.4 GB) 1030 -> 450 to 510 us by run and card
// -- 131 to 148 TFLOP/s, 168 to 190 with the columns' padding to 128; the
// splitting's vector instructions and the MFMAs, which share the issue slots,
// bound it at about 220 -- and a bf16 product of 96 x 96 blocks with 500
// columns (9.2 GFLOP) 128 -> 38 us.
//
// How an operand is loaded (chosen in the plan, a template parameter here):
//   K_RUN   k contiguous: a stage is [row][64 bytes of k]; the 16-byte granule
//           g of row r lies in slot g ^ ((r >> 2) & 3)
//   ROWS    rows contiguous: a stage is [k][rows]; fp32: granule g of row k in
//           slot g ^ 8 (k >> 3), bf16: in slot g ^ 4 ((k >> 1) & 1), read with
//           ds_read_b64_tr_b16 (one tile of rows: no swizzle)
//           Both copy 16 bytes per lane where rows, tiles and K are multiples
//           of 16 bytes, else 4: any fp32 size, even bf16 sizes.
//   K_ODD   bf16, k contiguous, rows on odd elements: straight to registers,
//           the aligned dwords around 8 k shifted by two bytes
//   GATHER  one element per load, its offset from the plan's tables (the k
//           table in LDS): more than one label in a role, odd bf16 rows
//   GATHER8 the same, eight k per load, where their offsets come in runs of
//           eight on whole dwords: 512 blocks of 64 x 256 with two contracted
//           labels apart, against 128 columns each, fp32 32.6 us (element
//           loads 49.8), bf16 19.7 (43.6)
// In the first three an element lies at row * sr + k * sk.
#include "lds_copy.h"
#include "split_f32.h"
#include "tre_internal.h"

#include <cmath>
#include <type_traits>

namespace tre {

namespace {

typedef split_f32x16 floatx16;
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(4))) int32_t const_i32;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

struct TileOp {
    const void* base;
    const int32_t* idx;  // tile index of each pair
    int64_t elems;
    const int32_t *tR, *tK, *tB;  // offsets of rows, k (both GATHER and GATHER8 only), batch
    int32_t rows, sr, sk;
    int32_t wide;  // K_RUN, ROWS: 16-byte copies (else 4)
};

struct TileArgs {
    TileOp a, b;
    int64_t w_elems;
    const int32_t *tWM, *tWN, *tWB;
    int32_t w_affine, w_sm;               // W(m, n) at m * w_sm + n
    int32_t batched;                      // several batch indices (their offsets from the tB tables)
    int32_t K, mblocks, nblocks, blocks;  // blocks: of one unit (batch x m x n)
    int32_t waves;                        // wavefronts per block: 4 or 1
    const Unit* units;
    const WsHeader* hdr;
    float* W;
    float* partials;
};

// k per chunk
template <typename T>
constexpr int kChunkK = sizeof(T) == 4 ? 16 : 32;

// The values of one chunk of one operand as a lane holds them: row l & 31 of
// each tile, k = 8 (l >> 5) .. + 7 of each 16.
template <typename T, int TT>
struct Raw {
    split_u32x4 v[2][TT];  // bf16 pairs: [16-k step][tile]
};
template <int TT>
struct Raw<float, TT> {
    float v[TT][8];
};

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// One operand of this wavefront's block, through LDS (K_RUN, ROWS).
template <typename T, int MODE, int TT>
struct Operand {
    static constexpr int E = int(sizeof(T));
    static constexpr int S = kChunkK<T> / 16;
    static constexpr bool kDma = true;
    static constexpr bool ROWS = MODE == TM_ROWS;
    static constexpr int kBytes = 2048 * TT;  // of a stage
    using R = Raw<T, TT>;
    uint32_t src[8 * TT];  // byte offsets of this lane's copies in a chunk (the first 2 TT when wide)
    uint32_t at;           // LDS offset of its fragments
    int64_t step;          // bytes per k of the chunk origin
    bool wide;
    int half;

    // slot of granule g in a [k][rows] stage
    static __device__ int swizzle(int k) {
        if (TT == 1) return 0;
        return E == 4 ? 8 * (k >> 3) : 4 * ((k >> 1) & 1);
    }
    __device__ void init(const TileOp& o, int r0, int K, const int32_t*) {
        const int lane = threadIdx.x & 63;
        half = lane >> 5;
        wide = o.wide;
        step = int64_t(ROWS ? o.sk : 1) * E;
        constexpr int kPitch = ROWS ? 32 * TT * E : 64;  // bytes of a stage row
        // copy q moves 64 x `bytes` consecutive bytes of the stage; the lane's
        // own start at `pos`
        auto source = [&](int q, int bytes) {
            const int pos = (q * 64 + lane) * bytes;
            const int line = pos / kPitch, slot = pos % kPitch / 16, in = pos % 16;
            if constexpr (ROWS) {
                const int k = min(line, K - 1), per = bytes / E;
                const int row = r0 + ((slot ^ swizzle(line)) * 16 + in) / E;
                return uint32_t(k * o.sk + min(row, o.rows - per)) * E;
            } else {
                const int k = ((slot ^ ((line >> 2) & 3)) * 16 + in) / E;
                return uint32_t(min(r0 + line, o.rows - 1) * o.sr + min(k, K - bytes / E)) * E;
            }
        };
#pragma unroll
        for (int q = 0; q < 8 * TT; q++) src[q] = wide && q < 2 * TT ? source(q, 16) : source(q, 4);
        const int r = lane & 31;
        if constexpr (!ROWS) at = uint32_t(r * 64);
        else if constexpr (E == 4) at = uint32_t(8 * half * kPitch + ((4 * r) ^ (TT == 2 ? 128 * half : 0)));
        else at = 0;
    }
    // copies of a chunk in flight
    __device__ int copies() const { return wide ? 2 * TT : 8 * TT; }
    // copy the chunk at k0 of the tile at `tile` (uniform) to the stage
    __device__ void copy(const char* tile, int k0, uint32_t stage) const {
        const char* p = tile + k0 * step;
        if (wide) {
#pragma unroll
            for (int q = 0; q < 2 * TT; q++) lds_copy16<false>(stage + q * 1024, p, src[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 8 * TT; q++) lds_copy4(stage + q * 256, p, src[q]);
        }
    }
    __device__ void read(R& x, const char* stage) const {
        const int lane = threadIdx.x & 63;
        if constexpr (!ROWS) {
            const int sw = (lane >> 2) & 3;
#pragma unroll
            for (int t = 0; t < TT; t++)
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    // fp32: the i-th half of the lane's 8 k; bf16: step i
                    const int g = E == 4 ? 2 * half + i : 2 * i + half;
                    const split_u32x4 d = *reinterpret_cast<const split_u32x4*>(stage + t * 2048 + at + ((g ^ sw) << 4));
                    if constexpr (E == 4) {
#pragma unroll
                        for (int j = 0; j < 4; j++) x.v[t][4 * i + j] = __uint_as_float(d[j]);
                    } else {
                        x.v[i][t] = d;
                    }
                }
        } else if constexpr (E == 4) {
#pragma unroll
            for (int t = 0; t < TT; t++)
#pragma unroll
                for (int j = 0; j < 8; j++)
                    x.v[t][j] = *reinterpret_cast<const float*>(stage + (at ^ (128 * t)) + j * (128 * TT));
        } else {
            const int i = lane & 15, G = lane >> 4;
            const int krow = 8 * (G >> 1) + (i >> 2);
#pragma unroll
            for (int t = 0; t < TT; t++) {
                const int gran = (4 * t + 2 * (G & 1) + ((i & 3) >> 1));
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    // (16 or 4 k-rows on, the swizzle is the same)
                    const char* p = stage + (krow + 16 * s) * (64 * TT) + ((gran ^ swizzle(krow)) << 4) + 8 * (i & 1);
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * (64 * TT)));
                    const s16x4 both[2] = {lo, hi};
                    x.v[s][t] = __builtin_bit_cast(split_u32x4, both);
                }
            }
        }
    }
};

// K_ODD, GATHER and GATHER8: straight to registers.
template <typename T, int MODE, int TT>
struct DirectOperand {
    static constexpr int E = int(sizeof(T));
    static constexpr int S = kChunkK<T> / 16;
    static constexpr bool kDma = false;
    static constexpr int kBytes = 0;
    using R = Raw<T, TT>;
    uint32_t ro[TT];  // byte offset of the lane's row (K_ODD: and its half's first k)
    int K;
    const int32_t* sK;  // GATHER, GATHER8: LDS k offsets
    int half;

    // rows r0 .. of the operand; rows past the end repeat the last one (their
    // results are never stored)
    __device__ void init(const TileOp& o, int r0, int K_, const int32_t* sK_) {
        const int lane = threadIdx.x & 63, r = lane & 31;
        half = lane >> 5;
        K = K_;
        sK = sK_;
#pragma unroll
        for (int t = 0; t < TT; t++) {
            const int row = min(r0 + 32 * t + r, o.rows - 1);
            if constexpr (MODE != TM_K_ODD) ro[t] = uint32_t(o.tR[row]) * E;
            else ro[t] = uint32_t(row * o.sr + 8 * half) * E;
        }
    }
    // the element of row offset `row` at contracted index k (clamped to K - 1;
    // values past the end are set to zero before the chunk is used)
    __device__ T element(const char* tile, uint32_t row, int k) const {
        return *reinterpret_cast<const T*>(tile + uint64_t(row + uint32_t(sK[min(k, K - 1)]) * E));
    }
    __device__ void load(R& x, const char* tile, int k0) const {
#pragma unroll
        for (int s = 0; s < S; s++)
#pragma unroll
            for (int t = 0; t < TT; t++) {
                if constexpr (MODE == TM_K_ODD) {
                    // the tile itself may start on an odd element
                    const uint32_t low = uint32_t(reinterpret_cast<uintptr_t>(tile)) & 2u;
                    const uint32_t o = ro[t] + uint32_t(k0 + 16 * s) * E + low, sh = o & 2u;
                    const char* p = tile - low + uint64_t(o & ~3u);
                    const u32x4u d = *reinterpret_cast<const u32x4u*>(p);
                    // the dword after, only read where it holds the eighth value
                    const uint32_t e = *reinterpret_cast<const uint32_t*>(p + 12 + 2 * sh);
                    x.v[s][t][0] = __builtin_amdgcn_alignbyte(d[1], d[0], sh);
                    x.v[s][t][1] = __builtin_amdgcn_alignbyte(d[2], d[1], sh);
                    x.v[s][t][2] = __builtin_amdgcn_alignbyte(d[3], d[2], sh);
                    x.v[s][t][3] = __builtin_amdgcn_alignbyte(e, d[3], sh);
                } else if constexpr (MODE == TM_GATHER8) {
                    // (K and the chunk's start are multiples of 8)
                    const uint32_t o = ro[t] + uint32_t(sK[min(k0 + 16 * s + 8 * half, K - 8)]) * E;
                    const u32x4u* p = reinterpret_cast<const u32x4u*>(tile + uint64_t(o));
                    const split_u32x4 lo = p[0];
                    if constexpr (E == 2) {
                        x.v[s][t] = lo;
                    } else {
                        const split_u32x4 hi = p[1];
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            x.v[t][j] = __uint_as_float(lo[j]);
                            x.v[t][4 + j] = __uint_as_float(hi[j]);
                        }
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        const T v = element(tile, ro[t], k0 + 16 * s + 8 * half + j);
                        if constexpr (E == 4) x.v[t][j] = v;
                        else if (j & 1) x.v[s][t][j >> 1] |= uint32_t(v) << 16;
                        else x.v[s][t][j >> 1] = v;
                    }
                }
            }
    }
};

template <typename T, int MODE, int TT>
using AnyOperand = std::conditional_t<MODE == TM_K_RUN || MODE == TM_ROWS, Operand<T, MODE, TT>, DirectOperand<T, MODE, TT>>;

// Before a chunk is used: zero its first `skip` k (taken by the chunk before)
// and those from `end` on (past K).
template <typename T, int TT>
__device__ inline void trim_chunk(Raw<T, TT>& x, int half, int skip, int end) {
#pragma unroll
    for (int s = 0; s < kChunkK<T> / 16; s++)
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int k = 16 * s + 8 * half + j;
            const bool keep = k >= skip && k < end;
#pragma unroll
            for (int t = 0; t < TT; t++)
                if constexpr (sizeof(T) == 4) x.v[t][j] = keep ? x.v[t][j] : 0.f;
                else x.v[s][t][j >> 1] &= keep ? 0xffffffffu : (j & 1) ? 0x0000ffffu : 0xffff0000u;
        }
}

// Chunks first, first + step, ... of a unit, pair by pair, `per` chunks each.
struct ChunkCursor {
    int p, q, per, step_p, step_q;
    __device__ void init(int p0, int first, int per_, int step) {
        per = per_;
        step_p = step / per;
        step_q = step % per;
        p = p0 + first / per;
        q = first % per;
    }
    __device__ void next() {
        q += step_q;
        const int wrap = q >= per ? 1 : 0;
        q -= wrap ? per : 0;
        p += step_p + wrap;
    }
};

template <typename T, int AM, int BM, int TM, int TN>
__global__ __launch_bounds__(kThreads, 2) void k_gemm_tile(TileArgs g) {
    using OpA = AnyOperand<T, AM, TM>;
    using OpB = AnyOperand<T, BM, TN>;
    constexpr bool kDma = OpA::kDma;
    static_assert(kDma == OpB::kDma, "both operands through LDS or neither");
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int KC = kChunkK<T>;
    constexpr int kStage = OpA::kBytes + OpB::kBytes;
    // [k tables of A, B][stages of the wavefronts, afterwards their sums]
    extern __shared__ __attribute__((aligned(1024))) float lds[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* sAK = reinterpret_cast<int32_t*>(lds);
    int32_t* sBK = sAK + g.K;
    constexpr bool kTables = AM == TM_GATHER || AM == TM_GATHER8;
    static_assert(kTables == (BM == TM_GATHER || BM == TM_GATHER8), "both operands through tables or neither");
    float* sums = lds + (kTables ? (2 * g.K + 3) / 4 * 4 : 0);  // (and stages: then no tables come before them)
    if constexpr (kTables) {
        for (int i = threadIdx.x; i < g.K; i += kThreads) {
            sAK[i] = g.a.tK[i];
            sBK[i] = g.b.tK[i];
        }
        __syncthreads();
    }
    // workgroups are dealt to the 8 XCDs in turn: the blocks of one unit take
    // consecutive places of one XCD and share its tiles in that L2
    const bool whole = g.waves == kWaves;  // the workgroup works on one block
    const int64_t xcd = blockIdx.x % 8, slot = int64_t(blockIdx.x / 8) * (whole ? 1 : kWaves) + (whole ? 0 : w);
    const int64_t unit_id = slot / g.blocks * 8 + xcd;
    int y = int(slot % g.blocks);
    if (unit_id >= g.hdr->n_units) return;
    const Unit un = g.units[unit_id];
    const int n0 = (y % g.nblocks) * 32 * TN;
    y /= g.nblocks;
    const int m0 = (y % g.mblocks) * 32 * TM;
    const int batch = y / g.mblocks;

    OpA oa;
    OpB ob;
    oa.init(g.a, m0, g.K, sAK);
    ob.init(g.b, n0, g.K, sBK);
    const char* Ab = reinterpret_cast<const char*>(g.a.base) + int64_t(g.batched ? g.a.tB[batch] : 0) * int(sizeof(T));
    const char* Bb = reinterpret_cast<const char*>(g.b.base) + int64_t(g.batched ? g.b.tB[batch] : 0) * int(sizeof(T));
    const int64_t a_bytes = g.a.elems * int(sizeof(T)), b_bytes = g.b.elems * int(sizeof(T));
    const const_i32* pa = (const const_i32*)g.a.idx;
    const const_i32* pb = (const const_i32*)g.b.idx;

    const int per = (g.K + KC - 1) / KC;
    const int total = (un.p1 - un.p0) * per;
    const int first = whole ? w : 0;
    const int n = total > first ? (total - first + g.waves - 1) / g.waves : 0;
    // start of chunk q inside the tile, and the k of it that count
    auto start = [&](int q) { return max(0, min(q * KC, g.K - KC)); };

    floatx16 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;
    };
    clear();
    // Loads run ahead of uses, and without a branch (where paths meet, values
    // still being loaded would be waited for): past the end they read the last
    // chunk again, which is never used.
    ChunkCursor cl, cu;  // the next chunk to load, the next to use
    int32_t ia, ib;      // tiles of the pair of cl, read ahead
    auto begin = [&]() {
        cl.init(un.p0, first, per, g.waves);
        cu = cl;
        ia = pa[cl.p];
        ib = pb[cl.p];
    };
    auto advance = [&]() {
        cl.next();
        const bool past = cl.p >= un.p1;
        cl.p = past ? un.p1 - 1 : cl.p;
        cl.q = past ? per - 1 : cl.q;
        ia = pa[cl.p];
        ib = pb[cl.p];
    };
    // through LDS: copy the next chunk to stage x, wait for the copies but
    // those of one chunk, read a stage
    char* stages = reinterpret_cast<char*>(sums) + w * (2 * kStage);
    const uint32_t stages_lds = __builtin_amdgcn_readfirstlane(lds_address(stages));
    auto copy = [&](int x) {
        if constexpr (kDma) {
            asm volatile("" : "+s"(ia), "+s"(ib));  // the indices are needed here, not where they were asked for
            const int k0 = start(cl.q);
            oa.copy(Ab + int64_t(ia) * a_bytes, k0, stages_lds + x * kStage);
            ob.copy(Bb + int64_t(ib) * b_bytes, k0, stages_lds + x * kStage + OpA::kBytes);
            advance();
        }
    };
    auto wait_one = [&]() {
        if constexpr (kDma) {
            if (oa.wide && ob.wide) lds_copy_wait<2 * (TM + TN)>();
            else if (oa.wide) lds_copy_wait<2 * TM + 8 * TN>();
            else if (ob.wide) lds_copy_wait<8 * TM + 2 * TN>();
            else lds_copy_wait<8 * (TM + TN)>();
        }
    };
    using RA = typename OpA::R;
    using RB = typename OpB::R;
    auto fetch = [&](int x, RA& ra, RB& rb) {  // a chunk's values: of stage x, or from memory
        if constexpr (kDma) {
            oa.read(ra, stages + x * kStage);
            ob.read(rb, stages + x * kStage + OpA::kBytes);
        } else {
            const int k0 = start(cl.q);
            oa.load(ra, Ab + int64_t(ia) * a_bytes, k0);
            ob.load(rb, Bb + int64_t(ib) * b_bytes, k0);
            advance();
        }
    };
    const bool trims = g.K % KC != 0;
    auto trim = [&](RA& ra, RB& rb) {
        const int k0 = start(cu.q), skip = cu.q * KC - k0, end = g.K - k0;
        trim_chunk<T, TM>(ra, oa.half, skip, end);
        trim_chunk<T, TN>(rb, ob.half, skip, end);
        cu.next();
    };
    float mx = 0.f;
    auto run = [&](auto with_trim) {
        constexpr bool kTrim = decltype(with_trim)::value;
        begin();
        copy(0);
        copy(1);
        if constexpr (F32) {
            // the splitting of a chunk runs between the MFMAs of the chunk
            // before, the copy of the chunk after next starts once the
            // stage's values are read
            RA ra;
            RB rb;
            Split8 fa[2][TM], fb[2][TN];
            wait_one();
            fetch(0, ra, rb);
            if constexpr (kTrim) trim(ra, rb);
            split_all(ra.v, rb.v, fa[0], fb[0], mx);
            lds_read_wait();
            copy(0);
            for (int i = 0; i + 1 < n; i += 2) {
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    wait_one();
                    fetch(1 - c, ra, rb);
                    if constexpr (kTrim) trim(ra, rb);
                    split_mma_next(acc, fa[c], fb[c], ra.v, rb.v, fa[1 - c], fb[1 - c], mx, [&] {
                        if constexpr (kDma) {
                            lds_read_wait();
                            copy(1 - c);
                        }
                    });
                }
            }
            if (n & 1) split_mma(acc, fa[0], fb[0]);
        } else {
            for (int i = 0; i < n; i += 2) {
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    if (c && i + 1 >= n) break;
                    RA ra;
                    RB rb;
                    wait_one();
                    fetch(c, ra, rb);
                    lds_read_wait();
                    copy(c);
                    if constexpr (kTrim) trim(ra, rb);
#pragma unroll
                    for (int s = 0; s < 2; s++)
#pragma unroll
                        for (int x = 0; x < TM; x++)
#pragma unroll
                            for (int z = 0; z < TN; z++)
                                acc[x][z] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    __builtin_bit_cast(split_bf16x8, ra.v[s][x]),
                                    __builtin_bit_cast(split_bf16x8, rb.v[s][z]), acc[x][z], 0, 0, 0);
                }
            }
        }
        // the copies past the end must land before the stages are used again
        if constexpr (kDma) lds_copy_wait<0>();
    };
    if (n > 0) {
        if (trims) run(std::true_type{});
        else run(std::false_type{});
    }

    // rows and columns of this lane's results
    const int col = lane & 31, half = lane >> 5;
    auto m_of = [&](int t, int r) {
        const int x = (r >> 2) * 8 + half * 4 + (r & 3);
        return m0 + 32 * t + x;
    };
    auto n_of = [&](int t) { return n0 + 32 * t + col; };
    float* out = un.slot < 0 ? g.W + int64_t(un.seg) * g.w_elems : g.partials + int64_t(un.slot) * g.w_elems;
    const int32_t ob_w = g.batched ? g.tWB[batch] : 0;
    // this wavefront's registers r0 .. r1 of every tile (all of them, or its
    // quarter after the sums over the wavefronts)
    int r0 = 0, r1 = 16;
    auto sum_waves = [&]() {
        // every wavefront leaves its sums (over the stages of all) and takes a
        // quarter of all of them
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM * TN; i++)
#pragma unroll
            for (int r = 0; r < 16; r++) sums[((w * TM * TN + i) * 16 + r) * 64 + lane] = acc[i / TN][i % TN][r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM * TN; i++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                float v = 0.f;
#pragma unroll
                for (int x = 0; x < kWaves; x++) v += sums[((x * TM * TN + i) * 16 + 4 * w + r) * 64 + lane];
                acc[i / TN][i % TN][r] = v;
            }
    };
    auto each = [&](auto f) {  // f(tile row, tile column, accumulator, its register number)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
#pragma unroll
                for (int r = 0; r < 16; r++)
                    if (r < r1 - r0) f(i, j, r, r0 + r);
    };
    if (whole) {
        sum_waves();
        r0 = 4 * w;
        r1 = r0 + 4;
    }
    if constexpr (F32) {
        SplitCheck check;
        each([&](int i, int j, int r, int reg) {
            if (m_of(i, reg) < g.a.rows && n_of(j) < g.b.rows) check.add(acc[i][j][r]);
        });
        bool redo;
        if (whole) {
            __syncthreads();  // the sums are read
            redo = split_bad_of_4(check, mx, sums);
            __syncthreads();
        } else {
            redo = split_bad(check, mx);
        }
        if (redo) {
            clear();
            if (n > 0) begin();
            for (int c = 0; c < n; c++) {
                RA ra;
                RB rb;
                copy(0);
                if constexpr (kDma) lds_copy_wait<0>();
                fetch(0, ra, rb);
                lds_read_wait();
                if (trims) trim(ra, rb);
#pragma unroll
                for (int s = 0; s < 8; s++)
#pragma unroll
                    for (int i = 0; i < TM; i++)
#pragma unroll
                        for (int j = 0; j < TN; j++)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ra.v[i][s], rb.v[j][s], acc[i][j], 0, 0, 0);
            }
            if (whole) sum_waves();
        }
    }
    if (g.w_affine) {
        float* at = out + ob_w;
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int m = m_of(i, r0 + r);
                if (r >= r1 - r0 || m >= g.a.rows) continue;
                float* row = at + int64_t(m) * g.w_sm;
#pragma unroll
                for (int j = 0; j < TN; j++) {
                    const int nn = n_of(j);
                    if (nn < g.b.rows) row[nn] = acc[i][j][r];
                }
            }
        return;
    }
    each([&](int i, int j, int r, int reg) {
        const int m = m_of(i, reg), nn = n_of(j);
        if (m < g.a.rows && nn < g.b.rows) out[ob_w + g.tWM[m] + g.tWN[nn]] = acc[i][j][r];
    });
}

template <typename T, int AM, int BM>
hipError_t dispatch_tiles(const Plan& p, const TileArgs& g, dim3 grid, size_t lds, hipStream_t s) {
    const dim3 block{unsigned(kThreads)};
    if (p.tile_m == 1)
        return p.tile_n == 1 ? launch_k(k_gemm_tile<T, AM, BM, 1, 1>, grid, block, lds, s, g)
                             : launch_k(k_gemm_tile<T, AM, BM, 1, 2>, grid, block, lds, s, g);
    return p.tile_n == 1 ? launch_k(k_gemm_tile<T, AM, BM, 2, 1>, grid, block, lds, s, g)
                         : launch_k(k_gemm_tile<T, AM, BM, 2, 2>, grid, block, lds, s, g);
}

template <typename T>
hipError_t dispatch(const Plan& p, const TileArgs& g, dim3 grid, size_t lds, hipStream_t s) {
    const int a = p.tile_op[0].mode, b = p.tile_op[1].mode;
    if (a == TM_GATHER)
        return b == TM_GATHER ? dispatch_tiles<T, TM_GATHER, TM_GATHER>(p, g, grid, lds, s)
                              : dispatch_tiles<T, TM_GATHER, TM_GATHER8>(p, g, grid, lds, s);
    if (a == TM_GATHER8)
        return b == TM_GATHER ? dispatch_tiles<T, TM_GATHER8, TM_GATHER>(p, g, grid, lds, s)
                              : dispatch_tiles<T, TM_GATHER8, TM_GATHER8>(p, g, grid, lds, s);
    if constexpr (sizeof(T) == 2)
        if (a == TM_K_ODD) return dispatch_tiles<T, TM_K_ODD, TM_K_ODD>(p, g, grid, lds, s);
    if (a == TM_K_RUN)
        return b == TM_K_RUN ? dispatch_tiles<T, TM_K_RUN, TM_K_RUN>(p, g, grid, lds, s)
                             : dispatch_tiles<T, TM_K_RUN, TM_ROWS>(p, g, grid, lds, s);
    return b == TM_K_RUN ? dispatch_tiles<T, TM_ROWS, TM_K_RUN>(p, g, grid, lds, s)
                         : dispatch_tiles<T, TM_ROWS, TM_ROWS>(p, g, grid, lds, s);
}

}  // namespace

// Time of a launch in microseconds, by rounds of the resident wavefronts (two
// workgroups of four on each of 256 CUs): `units` units of `chunks` chunks,
// `waves` wavefronts to a block.  A chunk of a wavefront takes about 1.2 us
// (fp32, both wavefronts of a SIMD busy) or 0.4 (bf16) for 2 x 2 MFMA tiles, a
// block's start and end about 6 (its dependent index and tile loads, the
// stores).
constexpr double kBlockTime = 6.0;
static double tile_blocks(const Plan& p) {
    const double M = double(p.swap ? p.nN : p.nM), N = double(p.swap ? p.nM : p.nN);
    return double(p.nB) * std::ceil(M / (32 * p.tile_m)) * std::ceil(N / (32 * p.tile_n));
}
static double chunk_time(const Plan& p) { return (p.dtype == TRE_BF16 ? 0.4 : 1.2) * p.tile_m * p.tile_n / 4.0; }
static double tile_time(const Plan& p, double units, double chunks, int waves) {
    const double slots = 512.0 * kWaves / waves;
    return std::ceil(units * tile_blocks(p) / slots) * (std::ceil(chunks / waves) * chunk_time(p) + kBlockTime);
}

// Unit length: keys are cut into c units each where that fills the chip's
// rounds better than it costs in partial tiles (written and read once, at
// about 4 TB/s, and one more launch).  On 320 keys of 256 pairs with two
// 64 x 64 blocks, one unit per key leaves 640 workgroups for 512 places, two
// rounds for the work of 1.25.  Where that does not pay, keys much longer than
// the average are still cut, so that none takes longer alone than the launch
// would with its work spread evenly, twice an average key or a block's start
// and end: of 401 keys one with 5,000 pairs of 32 x 48 tiles and the others
// with 2 took 1,905 us uncut.
int64_t tile_unit_pairs(const Plan& p, int64_t n_pairs, int64_t n_w) {
    const int64_t kc = p.dtype == TRE_BF16 ? kChunkK<uint16_t> : kChunkK<float>;
    const double per = double((p.nK + kc - 1) / kc), len = double(n_pairs) / double(std::max<int64_t>(n_w, 1));
    const int64_t whole = std::max<int64_t>(n_pairs, 1);
    if (n_w > 4096 || n_w < 1) return whole;
    double best = 0;
    int64_t unit = whole;
    for (int c = 1; c <= 64 && c <= len; c++) {
        const double pairs = std::ceil(len / c);
        const double t4 = tile_time(p, double(n_w) * c, pairs * per, kWaves), t1 = tile_time(p, double(n_w) * c, pairs * per, 1);
        double t = std::min(t4, t1);
        if (c > 1) t += 6.0 + double(n_w) * c * double(p.tile_elems[2]) * 8.0 / 4e6;
        if (c > 1 && t >= 0.95 * best) continue;
        best = t;
        unit = int64_t(pairs);
        if (c == 1) {
            const double waves = t1 < t4 ? 1 : kWaves;
            const double even = double(n_pairs) * tile_blocks(p) * waves / (512.0 * kWaves);
            const double block = 2 * kBlockTime * waves / (per * chunk_time(p));
            unit = int64_t(std::min(double(whole), std::ceil(std::max({2 * pairs, even, block}))));
        }
    }
    return unit;
}

hipError_t launch_gemm_tile(const Plan& p, const Layout& L, char* ws, const void* u_tiles, const void* v_tiles,
                            float* w_tiles, int64_t n_pairs, int64_t unit_bound, hipStream_t s) {
    const int32_t* tb = reinterpret_cast<const int32_t*>(ws + L.tables);
    const int32_t* pu = reinterpret_cast<const int32_t*>(ws + L.pu);
    const int32_t* pv = reinterpret_cast<const int32_t*>(ws + L.pv);
    TileArgs g{};
    auto operand = [&](TileOp& o, int x, const void* tiles, const int32_t* idx, int op, int tR, int tK, int tB,
                       int64_t rows) {
        o.base = tiles;
        o.idx = idx;
        o.elems = p.tile_elems[op];
        o.tR = tb + p.table_off[tR];
        o.tK = tb + p.table_off[tK];
        o.tB = tb + p.table_off[tB];
        o.rows = int32_t(rows);
        o.sr = p.tile_op[x].sr;
        o.sk = p.tile_op[x].sk;
        o.wide = p.tile_op[x].wide;
    };
    const int64_t M = p.swap ? p.nN : p.nM, N = p.swap ? p.nM : p.nN;
    operand(g.a, 0, p.swap ? v_tiles : u_tiles, p.swap ? pv : pu, p.swap ? 1 : 0, T_AM, T_AK, T_AB, M);
    operand(g.b, 1, p.swap ? u_tiles : v_tiles, p.swap ? pu : pv, p.swap ? 0 : 1, T_BN, T_BK, T_BB, N);
    g.w_elems = p.tile_elems[2];
    g.tWM = tb + p.table_off[T_WM];
    g.tWN = tb + p.table_off[T_WN];
    g.tWB = tb + p.table_off[T_WB];
    g.w_affine = p.tile_w_affine;
    g.w_sm = int32_t(p.tile_w_sm);
    g.batched = p.nB > 1;
    g.K = int32_t(p.nK);
    g.mblocks = int32_t((M + 32 * p.tile_m - 1) / (32 * p.tile_m));
    g.nblocks = int32_t((N + 32 * p.tile_n - 1) / (32 * p.tile_n));
    const int64_t blocks = p.nB * g.mblocks * g.nblocks;
    if (blocks > 65535) return hipErrorInvalidConfiguration;
    g.blocks = int32_t(blocks);
    g.units = reinterpret_cast<const Unit*>(ws + L.unit_desc);
    g.hdr = reinterpret_cast<const WsHeader*>(ws + L.hdr);
    g.W = w_tiles;
    g.partials = reinterpret_cast<float*>(ws + L.partials);
    // a wavefront or a workgroup per block, whichever the units' number and
    // length let finish first
    const int64_t kc = p.dtype == TRE_BF16 ? kChunkK<uint16_t> : kChunkK<float>;
    const double chunks = std::ceil(double(n_pairs) / double(unit_bound)) * double((p.nK + kc - 1) / kc);
    g.waves = tile_time(p, double(unit_bound), chunks, 1) < tile_time(p, double(unit_bound), chunks, kWaves) ? 1 : kWaves;
    const int64_t groups = (unit_bound + 7) / 8;  // units per XCD
    const int64_t per_wg = g.waves == 1 ? kWaves : 1;
    const int64_t grid = (groups * blocks + per_wg - 1) / per_wg * 8;
    if (grid > int64_t(0x7fffffff)) return hipErrorInvalidConfiguration;
    // the limit on the k tables is that of 64 + 64 + 2 K entries in 96 KB
    if (sizeof(int32_t) * size_t(128 + 2 * p.nK) > 96 * 1024) return hipErrorInvalidConfiguration;
    const bool gathered = p.tile_op[0].mode == TM_GATHER || p.tile_op[0].mode == TM_GATHER8;
    const size_t tables = gathered ? sizeof(int32_t) * size_t((2 * p.nK + 3) / 4 * 4) : 0;
    // a wavefront's two stages, or its sums
    const bool staged = p.tile_op[0].mode == TM_K_RUN || p.tile_op[0].mode == TM_ROWS;
    const size_t sums = kWaves * std::max<size_t>(staged ? 2 * 2048 * size_t(p.tile_m + p.tile_n) : 0,
                                                  g.waves == 1 ? 0 : sizeof(float) * size_t(p.tile_m * p.tile_n * 16 * 64));
    const dim3 gd{unsigned(grid), 1u, 1u};
    return p.dtype == TRE_BF16 ? dispatch<uint16_t>(p, g, gd, tables + sums, s)
                               : dispatch<float>(p, g, gd, tables + sums, s);
}

}  // namespace tre
