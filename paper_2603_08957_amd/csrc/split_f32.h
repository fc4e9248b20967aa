// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values, each the rest rounded
// to nearest even: x = h + m + l with |m| <= 2^-9 |x| and |l| <= 2^-18 |x|
// (24 significand bits, 8 per part).  A product is then the sum of nine exact
// bf16 products (16 bits each, exact in fp32); the three smallest (m l, l m,
// l l: together below 2^-26 of the product, a quarter of an fp32 rounding)
// are left out and six are added in fp32 by v_mfma_f32_32x32x16_bf16, the
// smallest first.  Six bf16 MFMAs of 32 cycles replace eight fp32 MFMAs of 64
// for the same 32x32x16 block, so the matrix cores need 192 instead of 512
// cycles; the splitting costs 6 vector instructions per element.
//
// Where the sum of the parts is not the value -- infinities, NaN, values that
// round to infinity, parts below bf16's smallest normal value 2^-126 -- the
// block is computed again by the fp32 MFMAs.  The kernels find that from
// results and from the largest input: an infinity or NaN in any input (or a
// part that became one) makes its results infinite or NaN; and with every
// |x| <= 2^30 a lost part (below 2^-126) changes a K-term sum by at most K
// 2^-96, less than 2^-24 of any result of at least 2^-50 for K up to 2^22.
// So a block is kept when no result is infinite or NaN, none lies strictly
// between 0 and 2^-50 and no input exceeds 2^30.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tre {

typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));
typedef float split_f32x16 __attribute__((ext_vector_type(16)));

constexpr float kSplitMaxInput = 0x1p30f;

// Eight values of one row as MFMA operands.
struct Split8 {
    split_u32x4 h, m, l;
    // values 2 i and 2 i + 1; `mx` collects the largest magnitude
    __device__ void set(int i, float x0, float x1, float& mx) {
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(mx) : "v"(x0), "v"(x1));
        const uint32_t hb = pack(x0, x1);
        const float r0 = x0 - __uint_as_float(hb << 16), r1 = x1 - __uint_as_float(hb & 0xffff0000u);
        const uint32_t mb = pack(r0, r1);
        h[i] = hb;
        m[i] = mb;
        l[i] = pack(r0 - __uint_as_float(mb << 16), r1 - __uint_as_float(mb & 0xffff0000u));
    }
    static __device__ uint32_t pack(float a, float b) {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(split_f32x2{a, b}, split_bf16x2));
    }
};

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
            if (f < TM) na[f].set(i, va[f][2 * i], va[f][2 * i + 1], mx);
            else nb[f - TM].set(i, vb[f - TM][2 * i], vb[f - TM][2 * i + 1], mx);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Collects whether every result lies where the split sum is as good as the
// fp32 one: 0, or finite and at least 2^-50.
struct SplitCheck {
    uint32_t top = 0, low = 0xffffffffu;
    __device__ void add(float v) {
        const uint32_t t = __float_as_uint(v) << 1;  // the magnitude's bits, doubled
        top = max(top, t);
        low = min(low, t - 1);  // zero wraps to the largest
    }
    __device__ bool bad(float max_input, float limit = kSplitMaxInput) const {
        constexpr uint32_t kInf2 = 0xff000000u, kMin2 = uint32_t(127 - 50) << 24;
        return top >= kInf2 || low < kMin2 - 1 || !(max_input <= limit);
    }
};

}  // namespace tre
