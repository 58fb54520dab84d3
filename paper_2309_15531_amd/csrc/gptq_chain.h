// What the two GPTQ sweeps (gptq_rows.h, gptq_groups.h) share: sizes, and the checks on the short quotients of their
// channel-by-channel chains.
//
// The length of the chain from one channel to the next is what a block's sweep takes, so the chains use short forms of
// the two quotients per channel and check beside the chain that these were right; a sub-block whose check fails is done
// again with plain divisions:
//   code   rint(w y) in place of rint(RN(w / s)), y within 2^-24 and a little of 1 / s: the same unless a half-way point
//          lies within 2^-22 |w y| of w y (w y is off by at most 2^-23 relative, RN(w / s) by 2^-24);
//   error  fastdiv's quotient of num = w - s k by d = U_ii, which fastdiv_corrected must leave as it is; num must be 0 or at
//          least 2^-80 for that correction to be exact, and 1/d RN (block_reciprocal; NaN outside fastdiv's range, which the
//          sweeps look for before they start a sub-block).
// NaN, infinities and quotients above 2^21 fail the first check, which so bounds w, num (s is at most 2^40) and the error.
// What was seen is kept as unsigned bit patterns (a compare per check would hold it in scalar registers, of which there are too few); with MASK
// the second check's outcome is a lane mask, one vector instruction less per channel where one row's chain leaves the registers for it
// (per IC, groups of 64, the mask costs 2.4 %: 512 x 2272 764 us and 783).
#pragma once

#include "common.h"
#include "fastdiv.h"

namespace {

namespace chain_ns {

constexpr int GB = 128;                // channels per block
constexpr int SB = 16;                 // channels per register sub-block of the chain
constexpr int PITCH = GB + 4;          // LDS row pitch (floats) of a strip and of the transposed block of U

template <bool MASK = false>
struct Check {
    uint32_t tie = 0u, off = 0u, num = 0xffffffffu;
    bool same = true;
    __device__ __forceinline__ void code(float quo, float near) {
        tie = max(tie, __float_as_uint(fmaf(fabsf(quo), 0x1p-22f, fabsf(quo - near))));
    }
    __device__ __forceinline__ void error(float n, float d, float y, float e) {
        if constexpr (MASK) same = same && fastdiv_corrected(n, d, y, e) == e;         // (false for a NaN, as without a reciprocal)
        else off |= __float_as_uint(fastdiv_corrected(n, d, y, e)) ^ __float_as_uint(e);
        num = min(num, (__float_as_uint(n) << 1) - 1u);       // zero wraps to the top
    }
    __device__ __forceinline__ bool fine() const {
        return tie <= 0x3F000000u && same && off == 0u && num >= (0x17800000u << 1) - 1u;      // 0.5, 2^-80
    }
};

__device__ __forceinline__ float block_reciprocal(float d) { return fastdiv_ok(d) ? 1.0f / d : __builtin_nanf(""); }
// whether all 16 reciprocals from rd on exist (whole wave)
__device__ __forceinline__ bool reciprocals_ok(const float* rd) {
    const float r = rd[threadIdx.x & (SB - 1)];
    return !__any(r != r);
}

// The value, recomputed from here on: address terms that do not change from block to block would otherwise be kept in
// registers over the whole sweep (or loop of work items), and there are more of them than registers.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ int fresh_uniform(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

}  // namespace chain_ns

}  // namespace
