// The per-IC GPTQ sweep: the walk over one 128-channel block, one launch per block (gfx950).  Included by gptq.hip.
//
// The parameters of (row group, channel) come from the channel's current values in all 64 or 128 rows of the group, so
// a group stays with one workgroup, and there are fewer groups than compute units: the errors' update of the columns
// behind the block is spread over the whole chip by launches of its own (gq_trailing).
//
// The walk: the strip sits in LDS, wave 0 takes 16 channels at a time into registers.  Its chain of decisions is what
// the block waits for: minimum and maximum of the group (one wave reduction), parameters, codes, errors, updates of
// the later channels of the sixteen.  Meanwhile the other waves apply the errors of the sixteen before to the
// columns behind; then all apply the new errors to the next sixteen columns.  Two error buffers, taken in turn.
// 128 rows: 55-61 us per block with eight waves where the chain with IEEE divisions and four waves took 76-78.
//
// Eight waves have all of a compute unit's registers, so no update runs beside them.  That is the faster form while the groups
// leave the update enough of the chip; beyond 160 groups four waves are.  us, eight / four waves (IEEE divisions and
// four waves): 64 groups of 64 x 1000 453 / 482 (657); 240 x 1000 817 / 759 (821); 272 x 2048 2979 / 2652
// (2852); 300 groups of 128 x 2048 5777 / 5202 (5712).  Up to 256 channels there is no update to leave room for, and eight are
// the faster form of any number: 389 groups of 64 x 256 201 / 211; 389 x 128 96 / 100.
//
// Registers: the form of 128 rows and eight waves spills 8, read back once per sub-block outside the chain.
//
// Every update is one rounded product and one rounded difference in channel order, whichever wave applies it.
// (Measured and not kept: the workgroup applying the last block's errors to its own strip first, which takes the launch
// between two sweeps out: 25 to 50 us of one compute unit's time against 10 to 19 of the chip's; and walk and update in
// one launch of 256 workgroups with a counter: the update then runs with the walk's registers at two waves per SIMD,
// half as fast, 270 us per block of an 11008-row layer against 185.)
#pragma once

#include "common.h"
#include "fastdiv.h"
#include "gptq_chain.h"
#include "scale_format.h"

namespace {

// Minima of two values over the wavefront, the same in every lane (min is exact, any order gives the
// same bits).  Butterflies inside the rows of 16 lanes, then row 0 into 1 and 2 into 3, then lane 31
// into the upper half, all as v_min_f32 with a DPP operand; lane 63 holds the result.  The two chains
// are interleaved and padded so that two wait states separate a write from the DPP read of it.
// Needs every lane active.
__device__ __forceinline__ void wave_min2(float& a, float& b) {
    asm volatile(
        "s_nop 1\n\t"
        "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_min_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 1"
        : "+v"(a), "+v"(b));
    a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 63));
    b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, b), 63));
}

namespace groups {

using namespace chain_ns;

constexpr int64_t MANY = 160;          // groups beyond which four waves walk a block that has updates beside it

template <int RPL>
struct Lds {
    float ut[GB][PITCH];               // ut[c][k] = U[i1 + k][i1 + c], the block's corner, transposed
    float w[64 * RPL][PITCH];          // the strip
    float es[2][SB][64 * RPL];         // errors of this sub-block and the last, [channel][row]
    float rd[GB];                      // 1 / U_ii of the block's channels (NaN: outside fastdiv's range)
};

struct QP {
    float scale, zero;
};
// the quantizer's parameters from a group's min and max (clip = 1): same formulas as adadim_quantize
// (mfmt != 0: the scale rounded into the 16-bit group word first, as adadim_quantize_meta16 does)
__device__ __forceinline__ QP params_of(float mn, float mx, float qmax, int mfmt) {
    mx = fmaxf(mx, 0.0f);
    mn = fminf(mn, 0.0f);
    const float range = mx - mn;
    float scale = range / qmax;
    if (range == 0.0f) scale = 1.0f;
    if (mfmt) scale = round_scale(scale, mfmt);
    float z = rintf((-mn) / scale);
    z = fminf(fmaxf(z, 0.0f), qmax);
    return {scale, z};
}

// Sub-block of 16 channels (n of them exist), rows l + 64 p in lane l.  FAST: the short quotients (gptq_chain.h); the
// reciprocal of the scale is v_rcp_f32 corrected once, the zero-point's quotient is checked like a code's, and
// range / qmax is fastdiv's, exact for ranges from 2^-60 up (2^-32 .. 2^40 is asked for here, which keeps the scale in
// fastdiv's range).  Returns false in a lane whose checks failed: nothing of the result is then to be used.
template <int RPL, bool FAST>
__device__ __forceinline__ bool chain(const float* w_lds, const float* ut, const float* rd, int n, float qmax, float rqmax, int mfmt,
                                      float (&e)[RPL][SB], uint32_t (&qpk)[RPL][SB / 4], float& my_scale, float& my_zero) {
    const int lane = threadIdx.x & 63;
    float w[RPL][SB];
#pragma unroll
    for (int p = 0; p < RPL; ++p) {
#pragma unroll
        for (int c = 0; c < SB; c += 4) {
            const float4 t = *reinterpret_cast<const float4*>(w_lds + (lane + 64 * p) * PITCH + c);
            w[p][c] = t.x; w[p][c + 1] = t.y; w[p][c + 2] = t.z; w[p][c + 3] = t.w;
        }
#pragma unroll
        for (int c = 0; c < SB / 4; ++c) qpk[p][c] = 0u;
    }
    Check check;
    uint32_t r_lo = 0xffffffffu, r_hi = 0u;                   // of the ranges (bit patterns; zero is allowed)
    // the corner of U (row cc of `ut` holds U[c][cc] for c <= cc) four columns at a time, two channels ahead of their use
    float ub[SB][SB], yd[SB];
    auto corner = [&](auto part_tag) {
        constexpr int C0 = decltype(part_tag)::value * 4;
#pragma unroll
        for (int cc = 0; cc < SB; ++cc) {
            if (cc >= C0) {
                const float4 t = *reinterpret_cast<const float4*>(ut + cc * PITCH + C0);
                ub[cc][C0] = t.x; ub[cc][C0 + 1] = t.y; ub[cc][C0 + 2] = t.z; ub[cc][C0 + 3] = t.w;
            }
        }
        const float4 t = *reinterpret_cast<const float4*>(rd + C0);
        yd[C0] = t.x; yd[C0 + 1] = t.y; yd[C0 + 2] = t.z; yd[C0 + 3] = t.w;
    };
    corner(std::integral_constant<int, 0>{});
#pragma unroll
    for (int c = 0; c < SB; ++c) {
        if ((c & 3) == 2 && c < 12) {
            asm volatile("" ::: "memory");                    // keeps these reads from moving up
            if (c == 2) corner(std::integral_constant<int, 1>{});
            if (c == 6) corner(std::integral_constant<int, 2>{});
            if (c == 10) corner(std::integral_constant<int, 3>{});
        }
        if (!FAST && c >= n) {                                // uniform
#pragma unroll
            for (int p = 0; p < RPL; ++p) e[p][c] = 0.0f;
            continue;
        }
        const float d = ub[c][c];
        float mn = w[0][c], nmx = -w[0][c];
#pragma unroll
        for (int p = 1; p < RPL; ++p) {
            mn = fminf(mn, w[p][c]);
            nmx = fminf(nmx, -w[p][c]);
        }
        wave_min2(mn, nmx);
        float scale, zero, y = 0.0f;
        if constexpr (FAST) {
            mn = fminf(mn, 0.0f);
            const float range = fmaxf(-nmx, 0.0f) - mn;
            scale = fastdiv(range, qmax, rqmax);
            r_lo = min(r_lo, __float_as_uint(range) - 1u);
            r_hi = max(r_hi, __float_as_uint(range));
            scale = range == 0.0f ? 1.0f : scale;
            if (mfmt) scale = round_scale(scale, mfmt);
            y = __builtin_amdgcn_rcpf(scale);
            y = fmaf(fmaf(-scale, y, 1.0f), y, y);
            const float zq = -mn * y, near = rintf(zq);
            check.code(zq, near);
            zero = __builtin_amdgcn_fmed3f(near, 0.0f, qmax);
        } else {
            const QP q = params_of(mn, -nmx, qmax, mfmt);
            scale = q.scale;
            zero = q.zero;
        }
        if (lane == c) {                                      // two selects; stored after the chain
            my_scale = scale;
            my_zero = zero;
        }
#pragma unroll
        for (int p = 0; p < RPL; ++p) {
            if constexpr (FAST) {
                const float quo = w[p][c] * y, near = rintf(quo);
                const float k = __builtin_amdgcn_fmed3f(near, -zero, qmax - zero);
                const float num = w[p][c] - scale * k;
                e[p][c] = fastdiv(num, d, yd[c]);
                qpk[p][c / 4] = __builtin_amdgcn_cvt_pk_u8_f32(k + zero, c & 3, qpk[p][c / 4]);
                check.code(quo, near);
                check.error(num, d, yd[c], e[p][c]);
            } else {
                float q = rintf(w[p][c] / scale) + zero;
                q = fminf(fmaxf(q, 0.0f), qmax);
                qpk[p][c / 4] |= static_cast<uint32_t>(q) << (8 * (c & 3));
                e[p][c] = (w[p][c] - scale * (q - zero)) / d;
            }
#pragma unroll
            for (int cc = 0; cc < SB; ++cc) {
                if (cc > c) {
                    const float upd = e[p][c] * ub[cc][c];
                    w[p][cc] = w[p][cc] - upd;
                }
            }
        }
    }
    return !FAST || (check.fine() && r_lo >= 0x2F800000u - 1u && r_hi <= 0x53800000u);   // 2^-32, 2^40
}

// Errors of the sub-block whose first channel is k0 (in the block), in `es`, applied to columns c and c + 1 of the
// strip (c even).  Channels that do not exist have error 0 and meet finite entries of `ut`.
template <int RPL>
__device__ __forceinline__ void apply2(const float (&e)[RPL][SB], const float* ut, float* w_lds, int k0, int c) {
    const int lane = threadIdx.x & 63;
    float u[2][SB];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < SB; k += 4) {
            const float4 q = *reinterpret_cast<const float4*>(ut + (c + t) * PITCH + k0 + k);
            u[t][k] = q.x; u[t][k + 1] = q.y; u[t][k + 2] = q.z; u[t][k + 3] = q.w;
        }
#pragma unroll
    for (int p = 0; p < RPL; ++p) {
        float2* at = reinterpret_cast<float2*>(w_lds + (lane + 64 * p) * PITCH + c);
        float2 v = *at;
#pragma unroll
        for (int k = 0; k < SB; ++k) {
            const float u0 = e[p][k] * u[0][k], u1 = e[p][k] * u[1][k];
            v.x = v.x - u0;
            v.y = v.y - u1;
        }
        *at = v;
    }
}

// Block [i1, i1 + nbw) of row group blockIdx.x.
template <int RPL, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void gq_group(const float* __restrict__ Wp, const float* __restrict__ U,
                                                          const int32_t* __restrict__ perm, int64_t in, int64_t i1, int nbw,
                                                          float qmax, float rqmax, int mfmt, float* __restrict__ scales_out,
                                                          uint8_t* __restrict__ zeros_out, uint8_t* __restrict__ Qp,
                                                          float* __restrict__ Ep) {
    constexpr int G = 64 * RPL;
    extern __shared__ __align__(16) char smem[];
    Lds<RPL>& lds = *reinterpret_cast<Lds<RPL>*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = int64_t(blockIdx.x) * G;
    const bool vec = (in & 3) == 0;                            // rows of Wp, Ep (scratch) start 16-byte aligned
    const bool vec_u = vec && (reinterpret_cast<uintptr_t>(U) & 15u) == 0;
    // four consecutive floats at src, of which n exist
    auto load4 = [](const float* src, int n, bool v4) {
        float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (v4 && n > 3) return *reinterpret_cast<const float4*>(src);
        if (n > 0) t.x = src[0];
        if (n > 1) t.y = src[1];
        if (n > 2) t.z = src[2];
        if (n > 3) t.w = src[3];
        return t;
    };
    {
        // The strip and the block's corner of U (transposed in LDS): 8 lanes along a row (one 128-byte line), RS rows at
        // a time, every load issued before the first value is stored.
        constexpr int RS = 8 * WAVES, NW = 4 * (G / RS), NU = 4 * (GB / RS);
        const int c4 = (tid & 7) * 4, kr = tid >> 3;
        float4 cu[NU], cw[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int r = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
            cw[q] = load4(Wp + (row0 + r) * in + i1 + c, nbw - c, vec);
        }
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int k = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
            cu[q] = k < nbw ? load4(U + (i1 + k) * in + i1 + c, nbw - c, vec_u) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        if (tid < GB) lds.rd[tid] = block_reciprocal(tid < nbw ? U[(i1 + tid) * (in + 1)] : 1.0f);
#pragma unroll
        for (int q = 0; q < NW; ++q) *reinterpret_cast<float4*>(&lds.w[kr + RS * (q >> 2)][c4 + 32 * (q & 3)]) = cw[q];
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int k = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
            lds.ut[c][k] = cu[q].x;
            lds.ut[c + 1][k] = cu[q].y;
            lds.ut[c + 2][k] = cu[q].z;
            lds.ut[c + 3][k] = cu[q].w;
        }
    }
    __syncthreads();

    for (int s0 = 0; s0 < nbw; s0 += SB) {
        const int sbw = min(nbw - s0, SB);
        float(*es)[G] = lds.es[(s0 / SB) & 1];
        if (wave == 0) {
            // the chain every later launch waits for: ahead of the bulk update that shares the SIMD with it
            __builtin_amdgcn_s_setprio(3);
            float e[RPL][SB], my_scale = 1.0f, my_zero = 0.0f;
            uint32_t qpk[RPL][SB / 4];
            const float* ut = &lds.ut[s0][s0];
            bool fine = sbw == SB && reciprocals_ok(&lds.rd[s0]);       // uniform
            if (fine) fine = chain<RPL, true>(&lds.w[0][s0], ut, &lds.rd[s0], SB, qmax, rqmax, mfmt, e, qpk, my_scale, my_zero);
            if (__any(!fine)) chain<RPL, false>(&lds.w[0][s0], ut, &lds.rd[s0], sbw, qmax, rqmax, mfmt, e, qpk, my_scale, my_zero);
            // the errors first: the other waves wait for them
#pragma unroll
            for (int p = 0; p < RPL; ++p)
#pragma unroll
                for (int k = 0; k < SB; ++k) es[k][lane + 64 * p] = e[p][k];
            if (lane < sbw) store_params(scales_out, zeros_out, int64_t(blockIdx.x) * in + perm[i1 + s0 + lane], my_scale, my_zero, mfmt);
            // codes and errors in visiting order
#pragma unroll
            for (int p = 0; p < RPL; ++p) {
                const int64_t at = (row0 + lane + 64 * p) * in + i1 + s0;
                if (sbw == SB && ((at & 15) == 0)) {
                    *reinterpret_cast<uint4*>(Qp + at) = make_uint4(qpk[p][0], qpk[p][1], qpk[p][2], qpk[p][3]);
                } else {
#pragma unroll
                    for (int c = 0; c < SB; ++c)
                        if (c < sbw) Qp[at + c] = static_cast<uint8_t>(qpk[p][c / 4] >> (8 * (c % 4)));
                }
                if (sbw == SB && vec) {
#pragma unroll
                    for (int c = 0; c < SB; c += 4)
                        *reinterpret_cast<float4*>(Ep + at + c) = make_float4(e[p][c], e[p][c + 1], e[p][c + 2], e[p][c + 3]);
                } else {
#pragma unroll
                    for (int c = 0; c < SB; ++c)
                        if (c < sbw) Ep[at + c] = e[p][c];
                }
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (s0 > 0 && s0 + SB < nbw) {
            // meanwhile the other waves bring the columns behind this sub-block up to date with the errors of the one
            // before it (this one's own columns got them ahead of the chain)
            const float(*el)[G] = lds.es[((s0 / SB) & 1) ^ 1];
            float e[RPL][SB];
#pragma unroll
            for (int p = 0; p < RPL; ++p)
#pragma unroll
                for (int k = 0; k < SB; ++k) e[p][k] = el[k][lane + 64 * p];
            for (int c = s0 + SB + 2 * (wave - 1); c < nbw; c += 2 * (WAVES - 1))
                apply2<RPL>(e, &lds.ut[0][0], &lds.w[0][0], s0 - SB, c);
        }
        if (s0 + SB >= nbw) break;                             // uniform: the last sub-block
        __syncthreads();
        // the new errors go to the next sub-block's columns at once, two or four for each wave, so that the chain can go on
        {
            float e[RPL][SB];
#pragma unroll
            for (int p = 0; p < RPL; ++p)
#pragma unroll
                for (int k = 0; k < SB; ++k) e[p][k] = es[k][lane + 64 * p];
#pragma unroll
            for (int c = 0; c < SB; c += 2 * WAVES) apply2<RPL>(e, &lds.ut[0][0], &lds.w[0][0], s0, s0 + SB + c + 2 * wave);
        }
        __syncthreads();
    }
}

template <int RPL, int WAVES>
hipError_t allow_lds_of() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gq_group<RPL, WAVES>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(sizeof(Lds<RPL>)));
}
inline hipError_t allow_lds() {
    for (const hipError_t e : {allow_lds_of<1, 4>(), allow_lds_of<1, 8>(), allow_lds_of<2, 4>(), allow_lds_of<2, 8>()})
        if (e != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace groups

}  // namespace
