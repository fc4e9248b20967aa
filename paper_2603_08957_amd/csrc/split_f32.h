// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values, each the rest rounded
// to nearest even: x = h + m + l with |m| <= 2^-8 |x| and |l| <= 2^-17 |x|
// (24 significand bits, 8 per part).  A product is then the sum of nine exact
// bf16 products (16 bits each, exact in fp32); the three smallest (m l, l m,
// l l: together at most 2^-24 of the product, one fp32 rounding, and 2^-27.5
// root mean square over random significands, where a rounding has 2^-25.3)
// are left out and six are added in fp32 by v_mfma_f32_32x32x16_bf16, the
// smallest first.  Six bf16 MFMAs of 32 cycles replace eight fp32 MFMAs of 64
// for the same 32x32x16 block, so the matrix cores need 192 instead of 512
// cycles; the splitting costs 6 vector instructions per element.
//
// Where the sum of the parts is not the value and that matters, the block is
// computed again by the fp32 MFMAs.  There are two such cases, each found where
// it arises:
//   the rest after h and m does not fit bf16: bits below 2^-133, which only
//     values below 2^-110 can have, so at most 2^-134 of a value is lost.  The
//     rests' lower 16 bits of a chunk (16 contracted indices) are collected in
//     the one instruction that this costs per two values; a chunk with such a
//     rest notes the largest value that it holds, M.  n products then change a
//     sum by at most n 2^-133 M, which is below 2^-24 of it where it is at
//     least 2^-88 M (n up to 2^21); a block with a smaller result runs again.
//   an infinity or NaN in an input, or a part or sum that became one: the
//     results that it enters are infinite or NaN.
// The conversions and the MFMAs keep subnormal parts, products and sums, so
// nothing else is lost, whatever the magnitudes: operands scaled by 1e-10 or
// 1e10 stay on the bf16 MFMAs, and so do ordinary sums with tiny terms (the
// tails of an exponential).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tre {

typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));
typedef float split_f32x16 __attribute__((ext_vector_type(16)));

// Eight values of one row as MFMA operands.
struct Split8 {
    split_u32x4 h, m, l;
    // values 2 i and 2 i + 1; the lower half of `lost` collects what their parts do not hold
    __device__ void set(int i, float x0, float x1, uint32_t& lost) {
        const uint32_t hb = pack(x0, x1);
        const float r0 = x0 - __uint_as_float(hb << 16), r1 = x1 - __uint_as_float(hb & 0xffff0000u);
        const uint32_t mb = pack(r0, r1);
        h[i] = hb;
        m[i] = mb;
        const float l0 = r0 - __uint_as_float(mb << 16), l1 = r1 - __uint_as_float(mb & 0xffff0000u);
        asm("v_or3_b32 %0, %1, %2, %0" : "+v"(lost) : "v"(l0), "v"(l1));
        l[i] = pack(l0, l1);
    }
    static __device__ uint32_t pack(float a, float b) {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(split_f32x2{a, b}, split_bf16x2));
    }
};

// Whether a lane's `lost` has anything, for the wavefront.
__device__ inline bool split_lost(uint32_t lost) { return __builtin_expect(__ballot((lost & 0xffffu) != 0) != 0, 0); }

// The largest magnitude (first part) of a fragment and m.
__device__ inline float split_largest(float m, const Split8& x) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        uint32_t h = x.h[i];
        asm("" : "+v"(h));  // unpacked here: the values unpacked for the rests would be kept until now
        m = fmaxf(m, fmaxf(fabsf(__uint_as_float(h << 16)), fabsf(__uint_as_float(h & 0xffff0000u))));
    }
    return m;
}

// A chunk's values as fragments; a chunk that loses something notes its
// largest value in `mx`.
template <int TM, int TN>
__device__ inline void split_note(uint32_t lost, const Split8 (&a)[TM], const Split8 (&b)[TN], float& mx) {
    if (!split_lost(lost)) return;
#pragma unroll
    for (int t = 0; t < TM; t++) mx = split_largest(mx, a[t]);
#pragma unroll
    for (int t = 0; t < TN; t++) mx = split_largest(mx, b[t]);
}

template <int TM, int TN>
__device__ inline void split_all(const float (&va)[TM][8], const float (&vb)[TN][8], Split8 (&a)[TM], Split8 (&b)[TN],
                                 float& mx) {
    uint32_t lost = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
#pragma unroll
        for (int t = 0; t < TM; t++) a[t].set(i, va[t][2 * i], va[t][2 * i + 1], lost);
#pragma unroll
        for (int t = 0; t < TN; t++) b[t].set(i, vb[t][2 * i], vb[t][2 * i + 1], lost);
    }
    split_note(lost, a, b, mx);
}

// acc[i][j] += A_i B_j over 16 contracted values (lane half h holds k = 8 h ..
// 8 h + 7 of its row in A and B), in kSplitSteps MFMAs, the smallest products
// first and the accumulators in turn.
template <int TM, int TN>
constexpr int kSplitSteps = 6 * TM * TN;

template <int TM, int TN>
__device__ inline void split_mma_step(int step, split_f32x16 (&acc)[TM][TN], const Split8 (&a)[TM],
                                      const Split8 (&b)[TN]) {
    const int q = step / (TM * TN), i = step % (TM * TN) / TN, j = step % TN;
    const split_u32x4 x = q == 0 ? a[i].l : (q == 2 || q == 3) ? a[i].m : a[i].h;
    const split_u32x4 y = q == 1 ? b[j].l : (q == 2 || q == 4) ? b[j].m : b[j].h;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(split_bf16x8, x),
                                                         __builtin_bit_cast(split_bf16x8, y), acc[i][j], 0, 0, 0);
}

template <int TM, int TN>
__device__ inline void split_mma(split_f32x16 (&acc)[TM][TN], const Split8 (&a)[TM], const Split8 (&b)[TN]) {
#pragma unroll
    for (int s = 0; s < kSplitSteps<TM, TN>; s++) split_mma_step(s, acc, a, b);
}

// The MFMAs of (a, b) with the splitting of the next fragments (raw values va,
// vb into na, nb) between them: a vector instruction issues while an MFMA
// runs, in one order that the compiler keeps, so a wavefront alone fills both.
// `mid` runs once the raw values are there.
template <int TM, int TN, typename Mid>
__device__ inline void split_mma_next(split_f32x16 (&acc)[TM][TN], const Split8 (&a)[TM], const Split8 (&b)[TN],
                                      const float (&va)[TM][8], const float (&vb)[TN][8], Split8 (&na)[TM],
                                      Split8 (&nb)[TN], float& mx, Mid mid) {
    uint32_t lost = 0;
    constexpr int kSteps = kSplitSteps<TM, TN>, kPairs = 4 * (TM + TN);
    constexpr int kLead = TM * TN;  // MFMAs that cover the latency of the raw values' reads
#pragma unroll
    for (int s = 0; s < kSteps; s++) {
        split_mma_step(s, acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
        if (s < kLead) continue;
        if (s == kLead) {
            mid();
            __builtin_amdgcn_sched_barrier(0);
        }
        const int p0 = (s - kLead) * kPairs / (kSteps - kLead), p1 = (s - kLead + 1) * kPairs / (kSteps - kLead);
#pragma unroll
        for (int p = p0; p < p1; p++) {
            const int f = p / 4, i = p % 4;
            if (f < TM) na[f].set(i, va[f][2 * i], va[f][2 * i + 1], lost);
            else nb[f - TM].set(i, vb[f - TM][2 * i], vb[f - TM][2 * i + 1], lost);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    split_note(lost, na, nb, mx);
}

// Whether a block's split sums stand.
struct SplitCheck {
    uint32_t top = 0, low = 0xffffffffu;  // the largest and smallest magnitude's bits, doubled
    __device__ void add(float v) {
        const uint32_t t = __float_as_uint(v) << 1;
        top = max(top, t);
        low = min(low, t);
    }
    __device__ bool infinite() const { return top >= 0xff000000u; }
    // a result that is not large beside what was lost (mx: the largest noted
    // value of all lanes, not 0)
    __device__ bool small(float mx) const { return low >> 1 < __float_as_uint(mx * 0x1p-88f); }
};

__device__ inline float split_wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// The verdict of a wavefront whose results only its own chunks enter; mx: what
// each lane noted.
__device__ inline bool split_bad(const SplitCheck& check, float mx) {
    bool bad = check.infinite();
    if (__ballot(mx > 0.f) != 0) bad = bad || check.small(split_wave_max(mx));
    return __ballot(bad) != 0;
}
// And of a workgroup of four whose results all their chunks enter; `shared`:
// eight floats of LDS that nothing else uses meanwhile.  Every wavefront gets
// the same answer.
__device__ inline bool split_bad_of_4(const SplitCheck& check, float mx, float* shared) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const float m = __ballot(mx > 0.f) != 0 ? split_wave_max(mx) : 0.f;
    const bool inf = __ballot(check.infinite()) != 0;
    if (lane == 0) {
        shared[w] = m;
        shared[4 + w] = inf ? 1.f : 0.f;
    }
    __syncthreads();
    const float all = fmaxf(fmaxf(shared[0], shared[1]), fmaxf(shared[2], shared[3]));
    bool bad = shared[4] + shared[5] + shared[6] + shared[7] != 0.f;
    if (all > 0.f && !bad) {  // (the same for all four)
        const bool small = __ballot(check.small(all)) != 0;
        __syncthreads();
        if (lane == 0) shared[w] = small ? 1.f : 0.f;
        __syncthreads();
        bad = shared[0] + shared[1] + shared[2] + shared[3] != 0.f;
    }
    return bad;
}

}  // namespace tre
