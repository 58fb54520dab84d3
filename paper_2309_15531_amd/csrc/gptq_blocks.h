// The per-OC GPTQ sweep with a launch per 128-channel block (gfx950), for the shapes that gptq_rows.h serves worse.
// Included by gptq.hip.
//
// A workgroup of four waves walks the block for 64 rows, twice as many as the widest workgroup of gptq_rows.h, and the
// errors' update of the channels behind the block is spread over the whole chip by launches of its own (gq_next,
// gq_trailing).  Which of the two forms a layer takes is launch_gptq_quantize's rule.
//
// Lane l of the first wave holds row 64 * block + l.  The rows live in an LDS strip; the channels are walked in sub-blocks
// of 16 that the first wave holds in registers: the sub-block's own updates stay in registers, then its 16 errors are
// posted in LDS.  All four waves apply them to the next sub-block's 16 columns at once, so that the chain can go on; the
// columns behind those receive them from the other three waves while the first one walks the next sub-block (two error
// buffers, taken in turn).  One LDS read and one write per element for 16 updates, always in channel order (which wave
// applies them does not change a bit).  The block of U is staged in LDS and read with wave-uniform addresses.
#pragma once

#include "common.h"
#include "gptq_chain.h"
#include "scale_format.h"

#include <type_traits>

namespace {

namespace blocks {

using chain_ns::GB;
using chain_ns::SB;

constexpr int ROWS = 64, PITCH = GB + 1;

struct Lds {
    float u[GB][GB];                                          // the block's corner of U
    float w[ROWS][PITCH];                                     // the strip
    float e[2][ROWS][SB + 1];                                 // errors of this sub-block and the last
};

// Block [i1, i1 + nbw).
__global__ __launch_bounds__(256) void gq_block(const float* __restrict__ Wp, const float* __restrict__ U,
                                               const int32_t* __restrict__ perm, int64_t out, int64_t in, int64_t i1, int nbw,
                                               int g, float qmax, int mfmt, const float* __restrict__ st_scales,
                                               const uint8_t* __restrict__ st_zeros, uint8_t* __restrict__ Qp,
                                               float* __restrict__ Ep) {
    extern __shared__ __align__(16) char smem[];
    Lds& lds = *reinterpret_cast<Lds*>(smem);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row0 = int64_t(blockIdx.x) * ROWS, row = row0 + lane;
    const bool ok = row < out;
    // The block of U and the strip of W: every thread's loads are issued before the first of them is stored, so the
    // block pays one trip to memory each, not one per loop iteration (16 and 32 of them: a fifth of the kernel).
    {
        constexpr int NU = GB * (GB / 4) / 256;               // 16-byte pieces of the block of U per thread
        float4 uv[NU];
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int e4 = threadIdx.x + 256 * q, k = e4 / (GB / 4), c4 = (e4 % (GB / 4)) * 4;
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k < nbw) {                                    // in % 4 == 0 is not required: guarded
                const float* src = U + (i1 + k) * in + i1 + c4;
                if (c4 + 3 < nbw && ((reinterpret_cast<uintptr_t>(src) & 15u) == 0)) {
                    v = *reinterpret_cast<const float4*>(src);
                } else {
                    if (c4 + 0 < nbw) v.x = src[0];
                    if (c4 + 1 < nbw) v.y = src[1];
                    if (c4 + 2 < nbw) v.z = src[2];
                    if (c4 + 3 < nbw) v.w = src[3];
                }
            }
            uv[q] = v;
        }
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int e4 = threadIdx.x + 256 * q, k = e4 / (GB / 4), c4 = (e4 % (GB / 4)) * 4;
            if (k < nbw) *reinterpret_cast<float4*>(&lds.u[k][c4]) = uv[q];
        }
    }
    {
        // consecutive lanes take consecutive columns
        constexpr int NR = ROWS / 2;
        const int c = threadIdx.x & (GB - 1), r_first = threadIdx.x >> 7;
        float wv[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int64_t r = row0 + r_first + 2 * j;
            wv[j] = (c < nbw && r < out) ? Wp[r * in + i1 + c] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (c < nbw) lds.w[r_first + 2 * j][c] = wv[j];
    }
    __syncthreads();
    const int n_cg = static_cast<int>(in / g);
    // errors of a sub-block applied to columns [c_lo, c_hi), every `step`-th from c_lo + first
    auto apply = [&](const float (*Esrc)[SB + 1], int k0, int kw, int c_lo, int c_hi, int first, int step) {
        float e[SB];
#pragma unroll
        for (int k = 0; k < SB; ++k) e[k] = Esrc[lane][k];
        for (int cc = c_lo + first; cc < c_hi; cc += step) {
            float u[SB];
#pragma unroll
            for (int k = 0; k < SB; ++k) u[k] = k < kw ? lds.u[k0 + k][cc] : 0.0f;
            if (!ok) continue;
            float v = lds.w[lane][cc];
#pragma unroll
            for (int k = 0; k < SB; ++k) {
                const float upd = e[k] * u[k];
                v = v - upd;
            }
            lds.w[lane][cc] = v;
        }
    };
    for (int s0 = 0; s0 < nbw; s0 += SB) {
        const int sbw = nbw - s0 < SB ? nbw - s0 : SB;
        float(*Es)[SB + 1] = lds.e[(s0 / SB) & 1];
        const float(*Es_last)[SB + 1] = lds.e[((s0 / SB) & 1) ^ 1];
        // the sequential part, one wave; FULL: all 16 channels exist (every sub-block but a ragged last one), which takes
        // the bounds tests and their branches out of the chain
        auto sub_block = [&](auto full_tag) {
            constexpr bool FULL = decltype(full_tag)::value;
            float w[SB], e[SB], scale[SB], zero[SB];
            uint32_t qpk[SB / 4];
#pragma unroll
            for (int c = 0; c < SB; ++c) w[c] = (ok && (FULL || c < sbw)) ? lds.w[lane][s0 + c] : 0.0f;
#pragma unroll
            for (int c = 0; c < SB / 4; ++c) qpk[c] = 0u;
            // the channels' original indices and static parameters: fetched together up front, off the chain
            int32_t jo[SB];
#pragma unroll
            for (int c = 0; c < SB; ++c) jo[c] = (FULL || c < sbw) ? perm[i1 + s0 + c] : 0;
#pragma unroll
            for (int c = 0; c < SB; ++c) {
                const bool have = ok && (FULL || c < sbw);
                if (mfmt) {                                   // static parameters as group words
                    const uint32_t wd = have ? reinterpret_cast<const uint16_t*>(st_scales)[row * n_cg + jo[c] / g]
                                             : (0x3C00u >> (mfmt - 1)) << mfmt;           // scale 1, zero 0
                    scale[c] = word_scale(wd, mfmt);
                    zero[c] = word_zero(wd, mfmt);
                } else {
                    scale[c] = have ? st_scales[row * n_cg + jo[c] / g] : 1.0f;
                    zero[c] = have ? static_cast<float>(st_zeros[row * n_cg + jo[c] / g]) : 0.0f;
                }
            }
            // The sub-block's 16 x 16 corner of U, all of it in registers before the chain starts (16-byte reads at
            // wave-uniform addresses): read row by row where it is used, each channel's chain began by waiting for its
            // row.  The fence keeps the reads up here.
            float ub[SB][SB];
#pragma unroll
            for (int c = 0; c < SB; ++c)
#pragma unroll
                for (int q4 = 0; q4 < SB / 4; ++q4) {
                    const float4 t = *reinterpret_cast<const float4*>(&lds.u[s0 + c][s0 + 4 * q4]);
                    ub[c][4 * q4 + 0] = t.x;
                    ub[c][4 * q4 + 1] = t.y;
                    ub[c][4 * q4 + 2] = t.z;
                    ub[c][4 * q4 + 3] = t.w;
                }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int c = 0; c < SB; ++c) {
                if (FULL || c < sbw) {                        // uniform
                    float q = rintf(w[c] / scale[c]) + zero[c];
                    q = fminf(fmaxf(q, 0.0f), qmax);
                    const float wq = scale[c] * (q - zero[c]);
                    qpk[c / 4] |= static_cast<uint32_t>(q) << (8 * (c % 4));
                    e[c] = (w[c] - wq) / ub[c][c];
                    // (constant bounds with a test, not "cc = c + 1": a trip count that depends on c is
                    // unrolled too late, after the loop has been vectorized with a run-time-indexed remainder)
#pragma unroll
                    for (int cc = 0; cc < SB; ++cc) {
                        if (cc > c && (FULL || cc < sbw)) {
                            const float upd = e[c] * ub[c][cc];
                            w[cc] = w[cc] - upd;
                        }
                    }
                } else {
                    e[c] = 0.0f;
                }
            }
            // the sub-block's codes and errors, in visiting order
            if (ok) {
                const int64_t at = row * in + i1 + s0;
                if (FULL && ((at & 15) == 0)) {
                    *reinterpret_cast<uint4*>(Qp + at) = make_uint4(qpk[0], qpk[1], qpk[2], qpk[3]);
                } else {
                    for (int c = 0; c < sbw; ++c) Qp[at + c] = static_cast<uint8_t>(qpk[c / 4] >> (8 * (c % 4)));
                }
                if (FULL && ((at & 3) == 0)) {
#pragma unroll
                    for (int c = 0; c < SB; c += 4)
                        *reinterpret_cast<float4*>(Ep + at + c) = make_float4(e[c], e[c + 1], e[c + 2], e[c + 3]);
                } else {
                    for (int c = 0; c < sbw; ++c) Ep[at + c] = e[c];
                }
            }
#pragma unroll
            for (int k = 0; k < SB; ++k) Es[lane][k] = e[k];
        };
        if (wave == 0) {
            // the chain every later launch waits for: ahead of the bulk update that shares the SIMD with it
            __builtin_amdgcn_s_setprio(3);
            if (sbw == SB) sub_block(std::true_type{});
            else sub_block(std::false_type{});
            __builtin_amdgcn_s_setprio(0);
        } else if (s0 > 0 && s0 + SB < nbw) {
            // meanwhile the other three waves bring the columns behind this sub-block up to date with the errors of the
            // sub-block before it (this sub-block's own columns got them ahead of the chain)
            apply(Es_last, s0 - SB, SB, s0 + SB, nbw, wave - 1, 3);
        }
        __syncthreads();
        // the new errors go to the next sub-block's columns at once, all four waves, so that the chain can go on
        if (s0 + SB < nbw) apply(Es, s0, sbw, s0 + SB, s0 + 2 * SB < nbw ? s0 + 2 * SB : nbw, wave, 4);
        __syncthreads();
    }
}

inline hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gq_block), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(sizeof(Lds)));
}

}  // namespace blocks

}  // namespace
