// The per-IC GPTQ sweep: one launch per 128-channel block (gfx950).  Included by gptq.hip.
//
// The parameters of (row group, channel) come from the channel's current values in all 64 or 128 rows of the group, so
// a group stays with one workgroup.  A block's launch holds two kinds of work that do not depend on each other, one workgroup
// of eight waves per compute unit taking them from one list:
//   * the walks, first in the list: a group's 128 columns get the last block's errors on their way from memory into LDS, then
//     its channels are visited one after the other;
//   * the update of the columns behind the block with the last block's errors, in pieces of 64 rows x 256 columns.
// Every element still receives the blocks' errors in block order, since a launch follows the one before it, and nothing
// else has to wait: no launch between two walks, no second stream, no event.  (The form before: the walk, a launch for the next
// block's columns, and the rest on a side stream, which the next block's launch had to wait for.  11008 x 4096, groups of
// 128: 60 + 17 us and 25 us of gaps per block beside updates of 210 to 20 us, 5260 us in all with the copies and the score; so
// 4650, the launches 230 us where 3840 columns are behind the block, 75 to 78 where few are.  More groups than compute units are
// no reason for the other form, with walks by four waves to leave the update room: us, launches of their own / one list, 172
// groups of 64 x 4096 4838 / 4352, 260 of 128 x 2048 4313 / 3582, 418 of 64 x 408 439 / 361, 1000 of 64 x 300 628 / 521; of 50
// sizes from 161 to 2000 groups 1.03 to 1.28 times as fast.)  Beyond the walks the update is
// bound by the pipes (3.0e13 elements per second of the 3.7e13 of gptq_update.h's bare loop).
//
// The walk: the strip sits in LDS, wave 0 takes 16 channels at a time into registers.  Its chain of decisions is what
// the block waits for: minimum and maximum of the group (one wave reduction), parameters, codes, errors, updates of
// the later channels of the sixteen.  Meanwhile the other waves apply the errors of the sixteen before to the
// columns behind; then all apply the new errors to the next sixteen columns.  Two error buffers, taken in turn.
// 128 rows, cycles of a block: strip 53000 (loads 9500, products and differences 37000), chains 84000, the rest 20000.
//
// Registers: with 128 rows 13 vector registers do not fit and live in scratch (56 bytes per lane), eleven of them read back once
// per sub-block behind the chain's short form, the others outside the loop over sub-blocks; with 64 rows none.  71 and 50 scalar
// ones live in lanes of vector registers.
//
// Every update is one rounded product and one rounded difference in channel order, whichever wave applies it.
#pragma once

#include "common.h"
#include "fastdiv.h"
#include "gptq_chain.h"
#include "gptq_update.h"
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

constexpr int WAVES = 8, ROWS = 64, COLS = 256;               // of a launch's workgroup; of a piece of the update

template <int RPL>
struct Walk {
    float ut[GB][PITCH];               // ut[c][k] = U[i1 + k][i1 + c], the block's corner, transposed
    float w[64 * RPL][PITCH];          // the strip
    float es[2][SB][64 * RPL];         // errors of this sub-block and the last, [channel][row]
    uint4 codes[2][64 * RPL];          // their codes, a row's sixteen
    float2 par[2][SB];                 // their scales and zero-points
    float rd[GB];                      // 1 / U_ii of the block's channels (NaN: outside fastdiv's range)
};

struct Piece {
    float es[2][ROWS][PITCH];          // errors of this piece's rows and the next's, [row][channel]
};
template <int RPL>
struct Lds {
    union {
        Walk<RPL> walk;
        Piece piece;
    };
    int taken;                         // next item of the list
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
    Check<> check;
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

// Four consecutive floats at src, of which n exist.
__device__ __forceinline__ float4 load4(const float* src, int n, bool v4) {
    float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (v4 && n > 3) return *reinterpret_cast<const float4*>(src);
    if (n > 0) t.x = src[0];
    if (n > 1) t.y = src[1];
    if (n > 2) t.z = src[2];
    if (n > 3) t.w = src[3];
    return t;
}

// The strip of a group: the columns [i1, i1 + nbw) of its rows with the errors of the block before (in Erows) applied.  The
// errors are staged where the strip will be; a wave takes 16 rows and 64 RPL columns.  Columns that do not exist become 0.
template <int RPL>
__device__ __forceinline__ void updated_strip(const float* __restrict__ Wrows, const float* __restrict__ U,
                                              const float* __restrict__ Erows, int64_t in64, int64_t i1, int nbw, bool vec,
                                              Walk<RPL>& lds) {
    constexpr int G = 64 * RPL, KB = 16, RS = 8 * WAVES, NE = 4 * (G / RS);
    const int tid = fresh(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const int rw = 16 * (RPL == 1 ? wave & 3 : wave), c0 = RPL == 1 ? 64 * (wave >> 2) : 0;
    const uint32_t pitch = 4u * static_cast<uint32_t>(in64);
    uint32_t ucol[RPL];
#pragma unroll
    for (int q = 0; q < RPL; ++q) ucol[q] = 4u * static_cast<uint32_t>(min(c0 + 64 * q + lane, nbw - 1));
    const update::Matrix W(Wrows + i1), Urows(U + (i1 - GB) * in64 + i1);
    float u[2][KB][RPL];
    auto fetch = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk)
#pragma unroll
            for (int q = 0; q < RPL; ++q) u[b][kk][q] = Urows.load(ucol[q], (k + kk) * pitch);
    };
    {
        const int c4 = (tid & 7) * 4, kr = tid >> 3;
        float4 ce[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) ce[q] = load4(Erows + (kr + RS * (q >> 2)) * in64 + c4 + 32 * (q & 3), 4, vec);
        fetch(0, 0);
#pragma unroll
        for (int q = 0; q < NE; ++q) *reinterpret_cast<float4*>(&lds.w[kr + RS * (q >> 2)][c4 + 32 * (q & 3)]) = ce[q];
    }
    update::f32x16 v[RPL], p[2];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < 4 * RPL; ++b)
            v[b >> 2][4 * (b & 3) + r] = W.load(static_cast<uint32_t>(rw + 4 * (lane >> 4)) * pitch +
                                                    4u * static_cast<uint32_t>(min(c0 + 16 * b + (lane & 15), nbw - 1)), r * pitch);
    __syncthreads();
    const float* e_row = &lds.w[rw + (lane & 15)][0];
    update::f32x4 ev[2];
    auto errors = [&](int b, int k) { ev[b] = *reinterpret_cast<const update::f32x4*>(e_row + (k & (GB - 1))); };
    errors(0, 0);
    p[0] = update::products16x64(ev[0].x, u[0][0][0]);
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
#pragma unroll
        for (int kk = 0; kk < 2 * KB; ++kk) {
            // (behind the block's last channel the first ones are read again and not used)
            if (kk == 0) fetch(1, k + KB);
            if (kk == KB) fetch(0, (k + 2 * KB) & (GB - 1));
            if ((kk & 3) == 0) errors(((kk >> 2) + 1) & 1, k + kk + 4);
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int at_q = kk * RPL + q, nq = (q + 1) % RPL, nk = q + 1 == RPL ? kk + 1 : kk;
                __builtin_amdgcn_sched_barrier(0);
                p[(at_q + 1) & 1] = update::products16x64(ev[(nk >> 2) & 1][nk & 3], u[(nk / KB) & 1][nk % KB][nq]);
                __builtin_amdgcn_sched_barrier(0);
                v[q] = v[q] - p[at_q & 1];
                asm volatile("" : "+v"(v[q]));                 // here, and not behind the next products
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < 4 * RPL; ++b) {
            const int c = c0 + 16 * b + (lane & 15);
            lds.w[rw + 4 * (lane >> 4) + r][c] = c < nbw ? v[b >> 2][4 * (b & 3) + r] : 0.0f;
        }
}

// Block [i1, i1 + nbw) of a row group, whose columns still lack the last block's errors.
template <int RPL>
__device__ __forceinline__ void walk(Walk<RPL>& lds, int group, const float* __restrict__ Wp, const float* __restrict__ U,
                                     const int32_t* __restrict__ perm, int64_t in, int64_t i1, int nbw, float qmax, float rqmax,
                                     int mfmt, float* __restrict__ scales_out, uint8_t* __restrict__ zeros_out,
                                     uint8_t* __restrict__ Qp, float* __restrict__ Ep) {
    constexpr int G = 64 * RPL;
    const int tid = fresh(threadIdx.x), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = int64_t(group) * G;
    const bool vec = (in & 3) == 0;                            // rows of Wp, Ep (scratch) start 16-byte aligned
    const bool vec_u = vec && (reinterpret_cast<uintptr_t>(U) & 15u) == 0;
    // The strip and the block's corner of U (transposed in LDS): 8 lanes along a row (one 128-byte line), RS rows at
    // a time, every load issued before the first value is stored.
    constexpr int RS = 8 * WAVES, NW = 4 * (G / RS), NU = 4 * (GB / RS);
    const int c4 = (tid & 7) * 4, kr = tid >> 3;
    float4 cu[NU];
    float cd = 1.0f;
    auto corner = [&] {
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int k = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
            cu[q] = k < nbw ? load4(U + (i1 + k) * in + i1 + c, nbw - c, vec_u) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        if (tid < nbw) cd = U[(i1 + tid) * (in + 1)];
    };
    if (i1 == 0) {
        float4 cw[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const int r = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
            cw[q] = load4(Wp + (row0 + r) * in + i1 + c, nbw - c, vec);
        }
        corner();
#pragma unroll
        for (int q = 0; q < NW; ++q) *reinterpret_cast<float4*>(&lds.w[kr + RS * (q >> 2)][c4 + 32 * (q & 3)]) = cw[q];
    } else {
        updated_strip<RPL>(Wp + row0 * in, U, Ep + row0 * in + i1 - GB, in, i1, nbw, vec, lds);
        corner();
    }
    if (tid < GB) lds.rd[tid] = block_reciprocal(cd);
#pragma unroll
    for (int q = 0; q < NU; ++q) {
        const int k = kr + RS * (q >> 2), c = c4 + 32 * (q & 3);
        lds.ut[c][k] = cu[q].x;
        lds.ut[c + 1][k] = cu[q].y;
        lds.ut[c + 2][k] = cu[q].z;
        lds.ut[c + 3][k] = cu[q].w;
    }
    __syncthreads();

    // A sub-block's codes, errors and parameters to memory, by the last waves: the rows lie far apart, and these stores would
    // hold up the chain by 3000 cycles per sub-block, next to its 10000.
    auto put_out = [&](int s0) {
        const int b = (s0 / SB) & 1, sbw = min(nbw - s0, SB), p = wave - (WAVES - RPL);
        if (wave == WAVES - 1 - RPL && lane < sbw) {
            const float2 t = lds.par[b][lane];
            store_params(scales_out, zeros_out, int64_t(group) * in + perm[i1 + s0 + lane], t.x, t.y, mfmt);
        }
        if (p < 0) return;
        const int64_t at = (row0 + lane + 64 * p) * in + i1 + s0;
        const uint4 q = lds.codes[b][lane + 64 * p];
        float e[SB];
#pragma unroll
        for (int c = 0; c < SB; ++c) e[c] = lds.es[b][c][lane + 64 * p];
        if (sbw == SB && (at & 15) == 0) {
            *reinterpret_cast<uint4*>(Qp + at) = q;
        } else {
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int c = 0; c < SB; ++c)
                if (c < sbw) Qp[at + c] = static_cast<uint8_t>(w[c / 4] >> (8 * (c % 4)));
        }
        if (sbw == SB && vec) {
#pragma unroll
            for (int c = 0; c < SB; c += 4) *reinterpret_cast<float4*>(Ep + at + c) = make_float4(e[c], e[c + 1], e[c + 2], e[c + 3]);
        } else {
#pragma unroll
            for (int c = 0; c < SB; ++c)
                if (c < sbw) Ep[at + c] = e[c];
        }
    };
    for (int s0 = 0; s0 < nbw; s0 += SB) {
        const int sbw = min(nbw - s0, SB);
        float(*es)[G] = lds.es[(s0 / SB) & 1];
        if (wave == 0) {
            // the chain the walk waits for: ahead of the wave that shares the SIMD with it
            __builtin_amdgcn_s_setprio(3);
            float e[RPL][SB], my_scale = 1.0f, my_zero = 0.0f;
            uint32_t qpk[RPL][SB / 4];
            const float* ut = &lds.ut[s0][s0];
            bool fine = sbw == SB && reciprocals_ok(&lds.rd[s0]);       // uniform
            if (fine) fine = chain<RPL, true>(&lds.w[0][s0], ut, &lds.rd[s0], SB, qmax, rqmax, mfmt, e, qpk, my_scale, my_zero);
            if (__any(!fine)) chain<RPL, false>(&lds.w[0][s0], ut, &lds.rd[s0], sbw, qmax, rqmax, mfmt, e, qpk, my_scale, my_zero);
#pragma unroll
            for (int p = 0; p < RPL; ++p) {
#pragma unroll
                for (int k = 0; k < SB; ++k) es[k][lane + 64 * p] = e[p][k];
                lds.codes[(s0 / SB) & 1][lane + 64 * p] = make_uint4(qpk[p][0], qpk[p][1], qpk[p][2], qpk[p][3]);
            }
            if (lane < SB) lds.par[(s0 / SB) & 1][lane] = make_float2(my_scale, my_zero);
            __builtin_amdgcn_s_setprio(0);
        } else if (s0 > 0) {
            put_out(s0 - SB);
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
        if (s0 + SB >= nbw) {                                  // uniform: the last sub-block
            __syncthreads();
            put_out(s0);
            break;
        }
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

// The pieces of the update of the columns [col0, in), errors of the block at k0, from item `first` of the list on (piece
// `item - n_groups`; a row of pieces after the other).  The next piece's errors, columns of W and first entries of U are on
// their way while a piece is worked on: with two waves per SIMD nothing else covers them.
__device__ __forceinline__ void pieces(Piece& lds, int* taken, int32_t* __restrict__ counter, int item, int n_groups, int n_items,
                                       float* __restrict__ Wp, const float* __restrict__ U, const float* __restrict__ Ep, int64_t in64,
                                       int64_t k0, int col0) {
    using update::row_of;
    constexpr int KB = 16, NE = ROWS * GB / 4 / (64 * WAVES);
    const int tid = threadIdx.x, lane = tid & 63, in = static_cast<int>(in64);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t pitch = 4u * static_cast<uint32_t>(in);
    const int per_row = (in - col0 + COLS - 1) / COLS;
    auto row0 = [&](int item) { return int64_t((item - n_groups) / per_row) * ROWS; };
    auto col = [&](int item) { return col0 + (item - n_groups) % per_row * COLS + 32 * wave; };    // the wave's first
    auto offset = [&](int item) { return 4u * static_cast<uint32_t>(min(col(item) + (lane & 31), in - 1)); };
    const uint32_t first = static_cast<uint32_t>(row_of(0, lane)) * pitch;
    const bool vec = (in & 3) == 0;                            // rows of Ep (scratch) start 16-byte aligned
    float4 eb[NE];
    auto load_errors = [&](int item) {
        const float* Erows = Ep + row0(item) * in64 + k0;
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int idx = tid + 64 * WAVES * q, r = idx / (GB / 4), k = idx % (GB / 4) * 4;
            eb[q] = load4(Erows + r * in64 + k, 4, vec);
        }
    };
    auto store_errors = [&](int b) {
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int idx = tid + 64 * WAVES * q, r = idx / (GB / 4), k = idx % (GB / 4) * 4;
            *reinterpret_cast<float4*>(&lds.es[b][r][k]) = eb[q];
        }
    };
    auto load = [&](int item, update::f32x32& v) {             // (past the last column: read, never stored)
        const update::Matrix Wrows(Wp + row0(item) * in64);
        const uint32_t off = first + offset(item);
#pragma unroll
        for (int r = 0; r < 32; ++r) v[r] = Wrows.load(off, row_of(r, 0) * pitch);
    };
    const update::Matrix Urows(U + k0 * in64);
    float u[2][KB];
    auto fetch = [&](int b, int k, uint32_t col) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) u[b][kk] = Urows.load(col, (k + kk) * pitch);
    };
    update::f32x32 v, v_next, p[2];
    uint32_t ucol = offset(item);
    load_errors(item);
    fetch(0, 0, ucol);
    load(item, v);
    store_errors(0);
    __syncthreads();
    for (int b = 0;; b ^= 1) {
        int ticket = 0;
        if (tid == 0) ticket = atomicAdd(counter, 1);
        const float* e_row = &lds.es[b][lane][0];
        update::f32x4 ev[2];
        auto errors = [&](int b, int k) { ev[b] = *reinterpret_cast<const update::f32x4*>(e_row + (k & (GB - 1))); };
        uint32_t ucol_next = ucol;
        const bool some = col(item) < in;                      // uniform: this wave has columns in the piece
        auto steps = [&](int k_begin) {
#pragma unroll 1
            for (int k = k_begin; k < k_begin + GB / 2; k += 2 * KB) {
                const uint32_t ucol2 = k + 2 * KB == GB ? ucol_next : ucol;    // behind the block's last channel: the next piece's first
#pragma unroll
                for (int kk = 0; kk < 2 * KB; ++kk) {
                    if (kk == 0) fetch(1, k + KB, ucol);
                    if (kk == KB) fetch(0, (k + 2 * KB) & (GB - 1), ucol2);
                    if ((kk & 3) == 0) errors(((kk >> 2) + 1) & 1, k + kk + 4);
                    const int nk = kk + 1;
                    __builtin_amdgcn_sched_barrier(0);
                    p[nk & 1] = update::products64x32(ev[(nk >> 2) & 1][nk & 3], u[(nk / KB) & 1][nk % KB]);
                    __builtin_amdgcn_sched_barrier(0);
                    v = v - p[kk & 1];
                    asm volatile("" : "+v"(v));                // here, and not behind the next products
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (some) {
            errors(0, 0);
            p[0] = update::products64x32(ev[0].x, u[0][0]);
            steps(0);
        }
        if (tid == 0) *taken = static_cast<int>(gridDim.x) + ticket;
        __syncthreads();
        const int next = __builtin_amdgcn_readfirstlane(*taken);
        const bool more = next < n_items;
        const int then = more ? next : item;                   // (none left: this one's are read again and not used)
        ucol_next = offset(then);
        load_errors(then);
        load(then, v_next);
        if (some) steps(GB / 2);
        else fetch(0, 0, ucol_next);
        store_errors(b ^ 1);
        if (col(item) + (lane & 31) < in) {
            const update::Matrix Wrows(Wp + row0(item) * in64);
            const uint32_t off = first + ucol;
#pragma unroll
            for (int r = 0; r < 32; ++r) Wrows.store(v[r], off, row_of(r, 0) * pitch);
        }
        if (!more) break;
        __syncthreads();
        item = then;
        ucol = ucol_next;
        v = v_next;
    }
}

// The launch of block [i1, i1 + nbw): items 0 .. n_groups - 1 are the groups' walks, the rest the pieces of the update.  A
// workgroup's first item is its own number, the later ones come from `counter` (0 at the start).
template <int RPL>
__global__ __launch_bounds__(64 * WAVES, 2) void gq_group_step(float* __restrict__ Wp, const float* __restrict__ U,
                                                         const int32_t* __restrict__ perm, int64_t in, int64_t i1, int nbw, int n_groups,
                                                         int n_items, float qmax, float rqmax, int mfmt, float* __restrict__ scales_out,
                                                         uint8_t* __restrict__ zeros_out, uint8_t* __restrict__ Qp,
                                                         float* __restrict__ Ep, int32_t* __restrict__ counter) {
    extern __shared__ __align__(16) char smem[];
    Lds<RPL>& lds = *reinterpret_cast<Lds<RPL>*>(smem);
    int item = static_cast<int>(blockIdx.x);
    while (item < n_groups) {
        walk<RPL>(lds.walk, item, Wp, U, perm, in, i1, nbw, qmax, rqmax, mfmt, scales_out, zeros_out, Qp, Ep);
        if (threadIdx.x == 0) lds.taken = static_cast<int>(gridDim.x) + atomicAdd(counter, 1);
        __syncthreads();                                       // (the walk's last reads of LDS are behind it, too)
        item = __builtin_amdgcn_readfirstlane(lds.taken);
        __syncthreads();
    }
    if (item < n_items) pieces(lds.piece, &lds.taken, counter, item, n_groups, n_items, Wp, U, Ep, in, i1 - GB, static_cast<int>(i1) + nbw);
}

// Pieces of the update in the launch of the block at i1 (none in the first one's).
inline int64_t n_pieces(int64_t out, int64_t in, int64_t i1) {
    const int64_t behind = i1 + GB;
    return i1 == 0 || behind >= in ? 0 : out / ROWS * ((in - behind + COLS - 1) / COLS);
}

template <int RPL>
hipError_t allow_lds_of() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gq_group_step<RPL>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(sizeof(Lds<RPL>)));
}
inline hipError_t allow_lds() {
    const hipError_t e = allow_lds_of<1>();
    return e == hipSuccess ? allow_lds_of<2>() : e;
}

}  // namespace groups

}  // namespace
