// The per-OC GPTQ sweep in one launch (gfx950).  Included by gptq.hip.
//
// With static groups (per-OC) the rows of W do not depend on each other, so a workgroup can take its R rows through
// every channel without meeting another workgroup.  While block b of 128 channels is walked, its eight waves do what they can of
// everything else:
//   * a chain wave per 16 rows walks the block: the rounding decisions, latency bound; helpers bring the block's later columns up to date
//     with each 16 channels' errors (chain_block, help_block);
//   * strips: the columns of block b + 1 get the errors of block b - 1 and then, as they come, those of block b, so that they are
//     finished as soon as the chain is; one more wave puts block b + 1's corner of U and its parameters where block b's have served;
//   * pieces of the columns behind block b + 1 get the errors of block b - 1 (a rounded product and a rounded
//     difference per element and channel, which is the definition's sequence, so no fma); everyone joins whose own work is done.
// One barrier per block; in between counters in LDS that only grow.  What bounds a block: its chain (10.4 us: about 600 instructions
// of one wave per 16 channels at 4 to 5 cycles each) where few columns are left or rows are few, else the update's arithmetic.  Whole calls, us,
// before (the step from block to block, 11 to 19 us, behind the chain, which took 12 to 23) and so: 512 x 1024 196 / 111, 256 x 4096 914 / 687,
// 2048 x 2048 507 / 439, 1000 x 272 65 / 38, 4096 x 4096 1751 / 1629 (bound by the update).
//
// Rows per workgroup: few enough that the chip's 256 compute units all have a workgroup (16 at 4096 rows), so that
// the update is spread over the whole chip; the chain takes much the same time for 4 rows as for 64.  rows_per_group
// picks R from the sizes.
//
// Registers: with 32 rows 8 vector registers do not fit and live in scratch, otherwise none.
//
// Order of the updates of one element: blocks in order, channels inside a block in order, whichever wave applies
// them; every update is one product and one difference.  Hence the same bits as a plain channel-by-channel loop.
#pragma once

#include "common.h"
#include "fastdiv.h"
#include "gptq_chain.h"
#include "gptq_update.h"
#include "scale_format.h"

#include <cmath>
#include <type_traits>

namespace {

namespace rows {

using namespace chain_ns;

constexpr int WAVES = 8;

// A workgroup's waves: one of the chain for up to 16 rows, then the chain's helpers, then those that are free.
template <int R>
constexpr int CHAINS = R <= 16 ? 1 : 2;
template <int R>
constexpr int HELPERS = R == 12 || R == 16 ? 2 : 1;             // per chain
template <int R>
constexpr int CR = R / CHAINS<R>;                               // rows of a chain
constexpr int pow2_rows(int r) { return r <= 4 ? 4 : r <= 8 ? 8 : 16; }

// Errors in LDS: [row][channel] where the matrix cores make the products (four channels of a row in one read), else
// [channel][row] (four rows of a channel).  Where channel c of row r is, and the words of a buffer.
template <int R>
constexpr bool BY_ROW = R == 16 || R == 32;
template <int R>
__device__ __forceinline__ constexpr int e_at(int c, int r) { return BY_ROW<R> ? r * PITCH + c : c * R + r; }
template <int R>
constexpr int E_WORDS = BY_ROW<R> ? R * PITCH : R * GB;

// LDS of one workgroup (dynamic)
template <int R>
struct Lds {
    float ut[GB][PITCH];               // ut[c][k] = U[i1 + k][i1 + c] for k < c, else 0: the block's corner, transposed
    float w[R][PITCH];                 // the block's columns of the rows, as the chain finds them
    float e[2][E_WORDS<R>];            // errors (e_at) of this block and the last
    float2 sc[GB][R];                  // static scale of (channel, row) and its reciprocal (NaN: outside fastdiv's range)
    float2 dg[GB];                     // U_ii of the block's channels and its reciprocal (NaN likewise)
    int cg[2][GB];                     // static group of the channels of this block and the next
    uint8_t zp[GB][R];                 // static zero-point
    int next[2];                       // next item of this block's list, and of the next one's
    int posted[CHAINS<R>], done[CHAINS<R> * HELPERS<R>];        // how far chains and helpers are (mark)
};

// Progress within a block, always growing: 16 blk + n.  A chain has posted n sub-blocks' errors; a helper has brought the
// sub-block n behind the first up to date with all before the one in front of it, and is through with the block at DONE.
constexpr int DONE = 15;
__device__ __forceinline__ constexpr int mark(int blk, int n) { return 16 * blk + n; }

// One wave tells others of its workgroup how far it is (everything it has put into LDS included), and they wait for that.
// Every wait of gq_rows ends: a chain waits only for what its helpers do with errors posted before, a helper only for its chain's
// next sub-block, and a strip for both, which start with the block, each in a wave of its own, and wait for no strip.
__device__ __forceinline__ void tell(int* count, int n) {
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(count, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wait_for(const int* count, int n) {
    while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) < n) {
    }
}

// lane i of each four (AGAIN: an instruction of its own; a bit without effect on lanes of four keeps the compiler from
// joining the two)
template <int I, bool AGAIN = false>
__device__ __forceinline__ float of_four(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x55 * I, 0xf, 0xf, !AGAIN));
}
// the value is worked out here, in the order of these calls
__device__ __forceinline__ void here(float& v) { asm volatile("" : "+v"(v)); }
template <typename F, int... I>
__device__ __forceinline__ void unrolled(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F f) {
    unrolled(f, std::make_integer_sequence<int, N>{});
}

// The same channel by channel in LDS with plain divisions: the ragged end of a row, and values outside the fast
// quotient's range.  n <= 16 channels; `par(c)` gives channel c's scale and zero-point, `put(c, code)` takes its code.
// Lanes that hold the same row do the same reads and writes in the same instruction.
template <int R, typename Par, typename Put>
__device__ __forceinline__ void chain_slow(float* wrow, const float* ut, const float2* dg, float* es_col, int n, float qmax, Par par, Put put) {
#pragma unroll 1
    for (int c = 0; c < n; ++c) {
        float sc, zp;
        par(c, sc, zp);
        const float w = wrow[c];
        float q = rintf(w / sc) + zp;
        q = fminf(fmaxf(q, 0.0f), qmax);
        put(c, static_cast<uint8_t>(q));
        const float e = (w - sc * (q - zp)) / dg[c].x;
        es_col[e_at<R>(c, 0)] = e;
#pragma unroll 1
        for (int cc = c + 1; cc < n; ++cc) {
            const float upd = e * ut[cc * PITCH + c];
            wrow[cc] = wrow[cc] - upd;
        }
    }
}

// One item of the update behind a block in vector instructions, for 4, 8 and 12 rows (24 as twice 12): columns c0 + lane + 64 q
// of RT of the workgroup's rows (Wrows and es point at the first of them), with the errors of the block at k0.  The products of
// update_behind make 16 rows whether they exist or not: 2618 x 8541 in twelves 6.19 ms so, 6.74 with them.  Matrix
// instructions of 4 rows x 64 columns would fit the rows, but eight of them and their differences take a SIMD 166 cycles for 2048
// elements, 64 of vector instructions 139 and one of 64 x 32 with its differences 134 (bare loops, two waves per SIMD);
// whether their fewer reads of the errors would make up for that was not tried.
// (offsets inside the workgroup's rows fit 32 bits: at most 32 rows of 46340)
template <int R, int RT, int CPL>
__device__ __forceinline__ void update_item(float* __restrict__ Wrows, const float* __restrict__ U, const float* es, int n_rows,
                                            int in_, int64_t k0, int c0) {
    // Channels per step: their entries of U travel one step ahead.  From memory that is a microsecond, which 64 of them in flight cover
    // (eight channels per step: 512 x 1024 in fours, 16 us per item).
    constexpr int KB = 64 / CPL;
    const int lane = fresh(threadIdx.x & 63), in = fresh_uniform(in_), c = c0 + CPL * lane;
    const uint32_t pitch = 4u * static_cast<uint32_t>(in), col = 4u * static_cast<uint32_t>(min(c, in - 1));
    const update::Matrix W(Wrows, int64_t(n_rows) * in), Urows(U + k0 * in, int64_t(in - k0) * in);
    float v[RT][CPL], u[2][KB][CPL];
    auto fetch = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) Urows.load(u[b][kk], col, (k + kk) * pitch);
    };
#pragma unroll
    for (int r = 0; r < RT; ++r) W.load(v[r], col, min(r, n_rows - 1) * pitch);      // past the end: read, never stored
    fetch(0, 0);
    // a channel's errors are read one channel ahead of their use, and no further (registers)
    float4 ev[2][RT / 4];
    auto errors = [&](int b, int k) {
#pragma unroll
        for (int i = 0; i < RT / 4; ++i) ev[b][i] = *reinterpret_cast<const float4*>(es + k * R + 4 * i);
    };
    auto step = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            errors((kk + 1) & 1, min(k + kk + 1, GB - 1));
#pragma unroll
            for (int i = 0; i < RT / 4; ++i) {
                const float4 e4 = ev[kk & 1][i];
                const float e[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < CPL; ++q) {
                        const float upd = e[j] * u[b][kk][q];
                        v[4 * i + j][q] = v[4 * i + j][q] - upd;
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int q = 0; q < CPL; ++q) here(v[r][q]);
    };
    errors(0, 0);
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
        fetch(1, k + KB);
        step(0, k);
        if (k + 2 * KB < GB) fetch(0, k + 2 * KB);
        step(1, k + KB);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        if (r >= n_rows) break;
        if (c + CPL <= in) {
            W.store(v[r], col, r * pitch);
        } else {
#pragma unroll
            for (int q = 0; q < CPL; ++q)
                if (c + q < in) W.store(v[r][q], col + 4 * q, r * pitch);
        }
    }
}

// The update behind a block for workgroups of 16 and 32 rows, the products on the matrix cores (gptq_update.h): items of 16
// rows x 64 NQ columns from column c_first on, as `take` gives them out, up to n_items; returns what it took last.  Two waves per SIMD keep the
// vector pipes busy only if neither waits for memory, so the next item's columns of W, and its first entries of U, are on
// their way while this one is worked on; and an instruction beside the differences costs a wave as much as one of them, so
// NQ products share a channel's errors and row of U, and four channels a read of the errors (64 columns and a read per
// channel: 90 us for 3712 columns, 83 with 128 and a read for four, before the last ones were halved).
template <int R, int NQ, typename Take>
__device__ __forceinline__ int update_behind(float* __restrict__ Wrows, const float* __restrict__ U, const float* es, int n_rows,
                                             int in_, int64_t k0, int c_first, int item, int n_items, Take take) {
    constexpr int RT = 16, COLS = 64 * NQ, KB = 8;             // KB channels per step: their U entries travel one step ahead
    const int lane = fresh(threadIdx.x & 63), in = fresh_uniform(in_);
    const uint32_t pitch = 4u * static_cast<uint32_t>(in);
    const update::Matrix W(Wrows), Urows(U + k0 * in);
    constexpr int HALVES = R / RT;
    // (the second half of a workgroup without so many rows: read and not stored)
    auto row0_of = [&](int item) { return HALVES == 1 ? 0 : (item & 1) * RT; };
    auto col0_of = [&](int item) { return c_first + (HALVES == 1 ? item : item >> 1) * COLS; };
    auto u_offset = [&](int item, int q) { return 4u * static_cast<uint32_t>(min(col0_of(item) + 64 * q + lane, in - 1)); };
    auto e_first = [&](int item) { return es + e_at<R>(0, row0_of(item) + (lane & 15)); };
    // past the last row or column: read, never stored
    auto load = [&](int item, update::f32x16 (&v)[NQ]) {
        const int rt = row0_of(item), c0 = col0_of(item);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t row = static_cast<uint32_t>(min(rt + 4 * (lane >> 4) + r, n_rows - 1)) * pitch;
#pragma unroll
            for (int b = 0; b < 4 * NQ; ++b)
                v[b >> 2][4 * (b & 3) + r] = W.load(row + 4u * static_cast<uint32_t>(min(c0 + 16 * b + (lane & 15), in - 1)), 0);
        }
    };
    float u[2][KB][NQ];
    auto fetch = [&](int b, int k, const uint32_t (&col)[NQ]) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk)
#pragma unroll
            for (int q = 0; q < NQ; ++q) u[b][kk][q] = Urows.load(col[q], (k + kk) * pitch);
    };
    update::f32x16 v[NQ], v_next[NQ], p[2];
    uint32_t ucol[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) ucol[q] = u_offset(item, q);
    const float* e_row = e_first(item);
    fetch(0, 0, ucol);
    load(item, v);
    update::f32x4 ev[2];
    ev[0] = *reinterpret_cast<const update::f32x4*>(e_row);
    p[0] = update::products16x64(ev[0].x, u[0][0][0]);
    for (;;) {
        const int taken = take();
        const bool more = taken < n_items;
        const int then = more ? taken : item;                  // (none left: this one's are read again and not used)
        uint32_t ucol_next[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) ucol_next[q] = u_offset(then, q);
        const float* e_next = e_first(then);
        auto steps = [&](int k_begin) {
#pragma unroll 1
            for (int k = k_begin; k < k_begin + GB / 2; k += 2 * KB) {
                const bool last = k + 2 * KB == GB;            // behind the block's last channel come the next item's first
                const float* e_behind = last ? e_next : e_row + k + 2 * KB;
                uint32_t ucol2[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) ucol2[q] = last ? ucol_next[q] : ucol[q];
#pragma unroll
                for (int kk = 0; kk < 2 * KB; ++kk) {
                    if (kk == 0) fetch(1, k + KB, ucol);
                    if (kk == KB) fetch(0, (k + 2 * KB) & (GB - 1), ucol2);
                    if ((kk & 3) == 0)
                        ev[((kk >> 2) + 1) & 1] = *reinterpret_cast<const update::f32x4*>(kk + 4 < 2 * KB ? e_row + k + kk + 4 : e_behind);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int at = kk * NQ + q, nk = q + 1 == NQ ? kk + 1 : kk, nq = (q + 1) % NQ;
                        __builtin_amdgcn_sched_barrier(0);
                        p[(at + 1) & 1] = update::products16x64(ev[(nk >> 2) & 1][nk & 3], u[(nk / KB) & 1][nk % KB][nq]);
                        __builtin_amdgcn_sched_barrier(0);
                        v[q] = v[q] - p[at & 1];
                        asm volatile("" : "+v"(v[q]));         // here, and not behind the next products
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        };
        steps(0);
        load(then, v_next);
        steps(GB / 2);
        {
            const int lane_s = fresh(lane), rt = row0_of(item), c0 = col0_of(item);
            const int rows_here = min(n_rows - rt, RT), cols_here = in - c0;
            const uint32_t first = static_cast<uint32_t>(4 * (lane_s >> 4)) * pitch + 4u * static_cast<uint32_t>(lane_s & 15);
            if (rows_here == RT && cols_here >= COLS) {        // uniform
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int b = 0; b < 4 * NQ; ++b) W.store(v[b >> 2][4 * (b & 3) + r], first, (rt + r) * pitch + 4 * (c0 + 16 * b));
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int b = 0; b < 4 * NQ; ++b)
                        if (4 * (lane_s >> 4) + r < rows_here && 16 * b + (lane_s & 15) < cols_here)
                            W.store(v[b >> 2][4 * (b & 3) + r], first, (rt + r) * pitch + 4 * (c0 + 16 * b));
            }
        }
        if (!more) return taken;
        item = then;
        e_row = e_next;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            ucol[q] = ucol_next[q];
            v[q] = v_next[q];
        }
    }
}

// The chain of a block, by one wave: CR rows (from r0 on) through its channels, 16 at a time.  Four lanes share a row: lane j holds the
// columns 4 t + j of a sub-block, t = 0 .. 3, and of the next one.  At channel 4 t + i all four work on their own column t, of
// which lane i's is the channel in turn: its error goes to the four by a DPP operand, and onto the columns that are left (`ut` is 0 for
// channels at and behind a column, which leaves a column that has had its turn as it is).  So behind channel 4 t + 3
// every lane holds its own column's decision, and the checks (gptq_chain.h) and codes cost a fourth of what they would for
// each channel in each lane.  The next sub-block's columns get the errors four channels late, which leaves the helpers time.
// With a lane per row, and sixteen columns
// in each, a channel took 37 instructions beside what followed the sub-block; so 26 with the next sub-block's columns.
template <int R>
__device__ __forceinline__ void chain_block(Lds<R>& lds, int ch, int blk, float* es, int n_rows, int nbw, float qmax,
                                            uint8_t* __restrict__ Qrows, int in) {
    constexpr int RR = pow2_rows(CR<R>);
    const int lane = fresh(threadIdx.x & 63), j = lane & 3, row_l = (lane >> 2) & (RR - 1);
    const bool row_in = row_l < CR<R>, first = lane < 4 * RR;               // (fewer than 16 rows: some lanes repeat others)
    const int crow = ch * CR<R> + (row_in ? row_l : 0);
    const bool row_ok = row_in && crow < n_rows, put_ok = row_ok && first;
    float* wrow = &lds.w[crow][0];
    uint8_t* q_row = Qrows + static_cast<uint32_t>(crow) * static_cast<uint32_t>(in);
    const bool words = (reinterpret_cast<uintptr_t>(Qrows) & 3u) == 0 && (in & 3) == 0;
    const int n_sub = (nbw + SB - 1) / SB;

    float w[4], wn[4], s[4], y[4], z[4], zq[4], d[4], yd[4], u[4][SB], un[4][SB];
    auto load_u = [&](int s0, int t, int q) {                // channels 4 q .. 4 q + 3 of column t
        const float4 v = *reinterpret_cast<const float4*>(&lds.ut[s0 + 4 * t + j][s0 + 4 * q]);
        u[t][4 * q] = v.x; u[t][4 * q + 1] = v.y; u[t][4 * q + 2] = v.z; u[t][4 * q + 3] = v.w;
    };
    auto load_par = [&](int s0, int t) {
        const int c = s0 + 4 * t + j;
        const float2 a = lds.sc[c][crow], b = lds.dg[c];
        s[t] = a.x; y[t] = a.y; d[t] = b.x; yd[t] = b.y;
        z[t] = static_cast<float>(lds.zp[c][crow]);
        zq[t] = qmax - z[t];
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        load_par(0, t);
#pragma unroll
        for (int q = 0; q <= t; ++q) load_u(0, t, q);
        w[t] = wrow[4 * t + j];
    }
#pragma unroll 1
    for (int sub = 0; sub < n_sub; ++sub) {
        const int s0 = sub * SB, sbw = min(nbw - s0, SB), s1 = min(s0 + SB, GB - SB);      // (behind the last: read and not used)
        const bool more = sub + 1 < n_sub;
        bool fine = sbw == SB;
        uint32_t pk = 0u;
        int ready[HELPERS<R>];
#pragma unroll
        for (int h = 0; h < HELPERS<R>; ++h)
            ready[h] = __hip_atomic_load(&lds.done[ch * HELPERS<R> + h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");                       // LDS serves a wave's reads in order: the counts first
#pragma unroll
        for (int t = 0; t < 4; ++t) wn[t] = wrow[s1 + 4 * t + j];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = *reinterpret_cast<const float4*>(&lds.ut[s1 + 4 * t + j][s0 + 4 * q]);
                un[t][4 * q] = v.x; un[t][4 * q + 1] = v.y; un[t][4 * q + 2] = v.z; un[t][4 * q + 3] = v.w;
            }
        // One wave's instruction that needs the one before it waits 9 cycles, any other 4 to 5: so each step of a channel's decision
        // is followed by its share of the work that waits for nothing: the last channel's error onto the later columns of the sub-block,
        // the one four channels back onto the next sub-block's, the last four's checks.
        float eb[SB], late_mul[3], next_mul[4];
        float quo[4], near[4], k[4], num[4], e[4];            // as the columns' decisions left them
        Check<true> check;
        auto besides = [&](auto c_tag, auto n_tag) {
            constexpr int C = decltype(c_tag)::value, N = decltype(n_tag)::value, T = C / 4, I = C % 4;
            if constexpr (N < 3) {                           // columns behind the one in turn: T + 1 .. 3
                if constexpr (C > 0 && T + N < 3) here(late_mul[N] = eb[C - 1] * u[T + 1 + N][C - 1]);
            } else if constexpr (N < 6) {
                if constexpr (C > 0 && T + N < 6) here(w[T + N - 2] = w[T + N - 2] - late_mul[N - 3]);
            } else if constexpr (N < 10) {
                if constexpr (T > 0) here(next_mul[N - 6] = eb[C - 4] * un[N - 6][C - 4]);
            } else if constexpr (N < 14) {
                if constexpr (T > 0) here(wn[N - 10] = wn[N - 10] - next_mul[N - 10]);
            } else {                                         // the four columns' decisions, each in its lane
                if constexpr (T > 0 && I == 0) {
                    if (row_in) es[e_at<R>(s0 + C - 4 + j, crow)] = e[T - 1];
                }
                if constexpr (T > 0 && I == 1) {
                    pk = __builtin_amdgcn_cvt_pk_u8_f32(k[T - 1] + z[T - 1], T - 1, pk);
                    check.code(quo[T - 1], near[T - 1]);
                }
                if constexpr (T > 0 && I == 2) check.error(num[T - 1], d[T - 1], yd[T - 1], e[T - 1]);
                if constexpr (T > 0 && I == 3) {
                    // the next sub-block's entries take the place of those that have served
                    load_par(s1, T - 1);
#pragma unroll
                    for (int t = T - 1; t < 4; ++t) load_u(s1, t, T - 1);
                }
            }
        };
        unrolled<SB>([&](auto c_tag) {
            constexpr int C = decltype(c_tag)::value, T = C / 4;
            if constexpr (C == 4) {
                if (sub > 0 && more) {
                    bool late = false;
#pragma unroll
                    for (int h = 0; h < HELPERS<R>; ++h) late |= __builtin_amdgcn_readfirstlane(ready[h]) < mark(blk, sub);
                    if (late) {
#pragma unroll
                        for (int h = 0; h < HELPERS<R>; ++h) wait_for(&lds.done[ch * HELPERS<R> + h], mark(blk, sub));
#pragma unroll
                        for (int t = 0; t < 4; ++t) wn[t] = wrow[s1 + 4 * t + j];
                    }
                }
            }
#define GQ_ASIDE(N) besides(c_tag, std::integral_constant<int, N>{})
            if constexpr (C > 0) {
                constexpr int I1 = (C - 1) % 4, T1 = (C - 1) / 4;
                float upd = of_four<I1>(e[T1]) * u[T][C - 1];
                here(upd);
                GQ_ASIDE(6);
                here(w[T] = w[T] - upd);
                here(eb[C - 1] = of_four<I1, true>(e[T1]));  // (again: the product above reads the four's lane by itself)
            }
            here(quo[T] = w[T] * y[T]);
            GQ_ASIDE(7);
            here(near[T] = rintf(quo[T]));
            GQ_ASIDE(8);
            GQ_ASIDE(0);
            // k = code - zero: clamping before or after the zero point is added is the same on integers
            here(k[T] = __builtin_amdgcn_fmed3f(near[T], -z[T], zq[T]));
            GQ_ASIDE(9);
            GQ_ASIDE(1);
            float sk = s[T] * k[T];
            here(sk);
            GQ_ASIDE(10);
            GQ_ASIDE(2);
            here(num[T] = w[T] - sk);
            GQ_ASIDE(11);
            GQ_ASIDE(3);
            float t0 = num[T] * yd[T];                        // fastdiv's steps
            here(t0);
            GQ_ASIDE(12);
            GQ_ASIDE(4);
            float r0 = fmaf(-d[T], t0, num[T]);
            here(r0);
            GQ_ASIDE(13);
            GQ_ASIDE(5);
            here(e[T] = fmaf(r0, yd[T], t0));
            GQ_ASIDE(14);
#undef GQ_ASIDE
        });
        eb[SB - 1] = of_four<3>(e[3]);
        if (row_in) es[e_at<R>(s0 + SB - 4 + j, crow)] = e[3];
        pk = __builtin_amdgcn_cvt_pk_u8_f32(k[3] + z[3], 3, pk);
        check.code(quo[3], near[3]);
        check.error(num[3], d[3], yd[3], e[3]);
        load_par(s1, 3);
        load_u(s1, 3, 3);
        auto onto_next = [&](int c) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float upd = eb[c] * un[t][c];
                wn[t] = wn[t] - upd;
            }
        };
        fine = fine && check.fine();
        if (!__any(row_ok && !fine)) {
            if (more) tell(&lds.posted[ch], mark(blk, sub + 1));
#pragma unroll
            for (int c = SB - 4; c < SB; ++c) onto_next(c);
            // codes in visiting order: lane j has those of the channels 4 t + j and stores 4 j .. 4 j + 3
            if (words) {
                uint32_t q = 0u;
                unrolled<4>([&](auto i_tag) {
                    constexpr int I = decltype(i_tag)::value;
                    const uint32_t v = __float_as_uint(of_four<I>(__uint_as_float(pk)));
                    q |= ((v >> (8 * j)) & 0xffu) << (8 * I);
                });
                if (put_ok) *reinterpret_cast<uint32_t*>(q_row + s0 + 4 * j) = q;
            } else if (put_ok) {
#pragma unroll
                for (int t = 0; t < 4; ++t) q_row[s0 + 4 * t + j] = static_cast<uint8_t>(pk >> (8 * t));
            }
        } else {
            // A channel at a time; the strip holds this sub-block's columns as they were.  (Lanes of a row do the same.)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (row_in) {
                chain_slow<R>(wrow + s0, &lds.ut[s0][s0], &lds.dg[s0], es + e_at<R>(s0, crow), sbw, qmax,
                              [&](int c, float& a, float& b) { a = lds.sc[s0 + c][crow].x; b = static_cast<float>(lds.zp[s0 + c][crow]); },
                              [&](int c, uint8_t q) { if (put_ok && j == 0) q_row[s0 + c] = q; });
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (more) {
                tell(&lds.posted[ch], mark(blk, sub + 1));
                if (sub > 0)
#pragma unroll
                    for (int h = 0; h < HELPERS<R>; ++h) wait_for(&lds.done[ch * HELPERS<R> + h], mark(blk, sub));
#pragma unroll
                for (int t = 0; t < 4; ++t) wn[t] = wrow[s1 + 4 * t + j];
#pragma unroll
                for (int c = 0; c < SB; ++c) {
                    eb[c] = es[e_at<R>(s0 + c, crow)];
                    onto_next(c);
                }
            }
        }
        if (more) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                wrow[s1 + 4 * t + j] = wn[t];                // (for chain_slow)
                w[t] = wn[t];
            }
        }
    }
    tell(&lds.posted[ch], mark(blk, n_sub));
}

// A chain's helper: a sub-block's errors onto the block's columns behind the next one, those behind that first.
template <int R>
__device__ __forceinline__ void help_block(Lds<R>& lds, int helper, int blk, const float* es, int nbw) {
    constexpr int RR = pow2_rows(CR<R>), CL = 64 / RR, NC = SB / (CL * HELPERS<R>);      // NC columns of a sub-block per lane
    const int lane = fresh(threadIdx.x & 63), ch = helper / HELPERS<R>, row_l = lane & (RR - 1);
    const int crow = ch * CR<R> + (row_l < CR<R> ? row_l : 0);
    const int cl = (lane / RR) + CL * NC * (helper % HELPERS<R>);
    float* wrow = &lds.w[crow][0];
    const int n_sub = (nbw + SB - 1) / SB;
#pragma unroll 1
    for (int sub = 0; sub + 2 < n_sub; ++sub) {
        const int s0 = sub * SB;
        wait_for(&lds.posted[ch], mark(blk, sub + 1));
        float e[SB];
#pragma unroll
        for (int k = 0; k < SB; ++k) e[k] = es[e_at<R>(s0 + k, crow)];
#pragma unroll 1
        for (int next = sub + 2; next < n_sub; ++next) {
            float v[NC], u[NC][SB];
#pragma unroll
            for (int t = 0; t < NC; ++t) {
                const int c = next * SB + cl + CL * t;
                v[t] = wrow[c];
#pragma unroll
                for (int k = 0; k < SB; k += 4) {
                    const float4 q = *reinterpret_cast<const float4*>(&lds.ut[c][s0 + k]);
                    u[t][k] = q.x; u[t][k + 1] = q.y; u[t][k + 2] = q.z; u[t][k + 3] = q.w;
                }
            }
#pragma unroll
            for (int k = 0; k < SB; ++k)
#pragma unroll
                for (int t = 0; t < NC; ++t) {
                    const float upd = e[k] * u[t][k];
                    v[t] = v[t] - upd;
                }
#pragma unroll
            for (int t = 0; t < NC; ++t) wrow[next * SB + cl + CL * t] = v[t];
            if (next == sub + 2) tell(&lds.done[helper], mark(blk, sub + 1));
        }
    }
    tell(&lds.done[helper], mark(blk, DONE));
}

// What a sub-block of the next block (at i2, whose groups are in cg) needs of U and the parameters: fetched ahead by one wave, put into
// LDS where this block no longer needs its own.
template <int R>
struct Stage {
    static constexpr int NP = SB * R / 64;                     // parameters per lane
    float u[2][SB], ps[NP], pz[NP], d;                         // u[q][k]: column lane + 64 q

    __device__ __forceinline__ void fetch(const float* __restrict__ U, int in, int i2, int nbw, int sub, const int* cg, int64_t row0,
                                          int n_rows, int n_cg, int mfmt, const float* __restrict__ st_scales,
                                          const uint8_t* __restrict__ st_zeros) {
        const int lane = fresh(threadIdx.x & 63), s0 = sub * SB;
        const uint32_t pitch = 4u * static_cast<uint32_t>(in);
        const update::Matrix corner(U + int64_t(i2) * in + i2);
        // (past the end of the last block: read again, and met by no error)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t col = 4u * static_cast<uint32_t>(min(lane + 64 * q, nbw - 1));
#pragma unroll
            for (int k = 0; k < SB; ++k) u[q][k] = corner.load(col, static_cast<uint32_t>(min(s0 + k, nbw - 1)) * pitch);
        }
        d = corner.load(static_cast<uint32_t>(min(s0 + (lane & 15), nbw - 1)) * (pitch + 4u), 0);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int idx = lane + 64 * q, c = s0 + idx / R, r = idx % R;
            const int64_t at = (row0 + min(r, n_rows - 1)) * n_cg + cg[c];
            if (mfmt) {
                ps[q] = __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(st_scales)[at]));
                pz[q] = 0.0f;
            } else {
                ps[q] = st_scales[at];
                pz[q] = static_cast<float>(st_zeros[at]);
            }
        }
    }
    __device__ __forceinline__ void put(Lds<R>& lds, int sub, int mfmt) const {
        const int lane = fresh(threadIdx.x & 63), s0 = sub * SB;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < SB; k += 4) {
                const int c = lane + 64 * q;
                auto above = [&](int i) { return s0 + k + i < c ? u[q][k + i] : 0.0f; };
                *reinterpret_cast<float4*>(&lds.ut[c][s0 + k]) = make_float4(above(0), above(1), above(2), above(3));
            }
        if (lane < SB) lds.dg[s0 + lane] = make_float2(d, block_reciprocal(d));
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int idx = lane + 64 * q, c = s0 + idx / R, r = idx % R;
            float sc = ps[q], zp = pz[q];
            if (mfmt) {                                        // ps holds the group word's bits
                const uint32_t wd = __float_as_uint(sc);
                sc = word_scale(wd, mfmt);
                zp = word_zero(wd, mfmt);
            }
            lds.sc[c][r] = make_float2(sc, fastdiv_ok(sc) ? 1.0f / sc : __builtin_nanf(""));
            lds.zp[c][r] = static_cast<uint8_t>(zp);
        }
    }
};

// A strip of the next block's columns: four columns and RQ rows per lane.
template <int R>
struct Strip {
    static constexpr int COLS = R == 4 ? 64 : 32, CL = COLS / 4, RQ = (R * CL + 63) / 64, COUNT = GB / COLS;
    float v[RQ][4];

    static __device__ __forceinline__ int row(int lane, int r) { return min(lane / CL * RQ + r, R - 1); }      // (the last ones repeat)

    // Errors of the sixteen channels from k0 on (e_at) onto the columns: a product and a difference each.
    __device__ __forceinline__ void apply(const float* es, int k0, int lane, const float (&u)[SB][4]) {
#pragma unroll
        for (int k = 0; k < SB; k += 4) {
            float e[4][RQ];
#pragma unroll
            for (int r = 0; r < RQ; ++r) {
                if constexpr (BY_ROW<R>) {
                    const float4 t = *reinterpret_cast<const float4*>(es + e_at<R>(k0 + k, row(lane, r)));
                    e[0][r] = t.x; e[1][r] = t.y; e[2][r] = t.z; e[3][r] = t.w;
                } else {
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) e[kk][r] = es[e_at<R>(k0 + k + kk, row(lane, r))];
                }
            }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int r = 0; r < RQ; ++r)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float upd = e[kk][r] * u[k + kk][q];
                        v[r][q] = v[r][q] - upd;
                    }
            __builtin_amdgcn_sched_barrier(0);
        }
        // here, and not behind the next wait, where this one's entries of U would still be held
#pragma unroll
        for (int r = 0; r < RQ; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) here(v[r][q]);
    }
};

template <int R>
__global__ __launch_bounds__(64 * WAVES, 2) void gq_rows(float* __restrict__ Wp, const float* __restrict__ U,
                                                         const int32_t* __restrict__ perm, int64_t out, int64_t in64, int g,
                                                         float qmax, int mfmt, const float* __restrict__ st_scales,
                                                         const uint8_t* __restrict__ st_zeros, uint8_t* __restrict__ Qp) {
    // items of the update: RT rows x 128 columns on the matrix cores where RT is 16, else RT rows x 64 CPL columns (RT x CPL
    // accumulators; few rows take more columns, so that an LDS read of the errors serves as many products)
    constexpr int CPL = R <= 8 ? 4 : 2, RT = R <= 16 ? R : R / 2, ITEM = RT == 16 ? 128 : 64 * CPL;
    constexpr int HELPERS_ALL = CHAINS<R> * HELPERS<R>;
    constexpr int PIECES_AT = 1 + Strip<R>::COUNT;             // the first piece of the update in a block's list
    constexpr int NARROW = R == 16 ? 14 : 4;                   // pieces cut in two
    extern __shared__ __align__(16) char smem[];
    Lds<R>& lds = *reinterpret_cast<Lds<R>*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = int64_t(blockIdx.x) * R;
    const int n_rows = static_cast<int>(min(out - row0, int64_t(R)));        // > 0
    const int in = static_cast<int>(in64), n_cg = in / g;
    float* __restrict__ Wrows = Wp + row0 * in64;

    // static groups of the channels of the block at i1
    auto stage_groups = [&](int i1, int* cg) {
        for (int c = fresh(threadIdx.x & 63); c < GB; c += 64)
            cg[c] = i1 + c < in ? static_cast<int>(static_cast<uint32_t>(perm[i1 + c]) / static_cast<uint32_t>(g)) : 0;
    };

    // first block: its columns straight into the strip; a wave per sub-block for the rest
    if (wave < 2) stage_groups(GB * wave, lds.cg[wave]);
    if (tid < 2) lds.next[tid] = 0;
    if (tid < CHAINS<R>) lds.posted[tid] = 0;
    if (tid < HELPERS_ALL) lds.done[tid] = 0;
    __syncthreads();
    {
        const int nbw = min(in, GB);
        for (int idx = tid; idx < R * GB; idx += 64 * WAVES) {
            const int r = idx / GB, c = idx % GB;
            lds.w[r][c] = (c < nbw && r < n_rows) ? Wrows[static_cast<uint32_t>(r) * static_cast<uint32_t>(in) + c] : 0.0f;
        }
        Stage<R> st;
        st.fetch(U, in, 0, nbw, wave, lds.cg[0], row0, n_rows, n_cg, mfmt, st_scales, st_zeros);
        st.put(lds, wave, mfmt);
    }
    __syncthreads();

    for (int i1 = 0, blk = 0; i1 < in; i1 += GB, ++blk) {
        const int nbw = min(in - i1, GB), behind = i1 + nbw;
        float* es = lds.e[blk & 1];
        const float* es_last = lds.e[(blk & 1) ^ 1];
        const int next_w = min(in - behind, GB), far = behind + GB;          // (the next block's width, if there is one)
        if (wave < CHAINS<R>) {
            // the chain the workgroup waits for: ahead of the updates that share its SIMD
            __builtin_amdgcn_s_setprio(3);
            chain_block<R>(lds, wave, blk, es, n_rows, nbw, qmax, Qp + row0 * in64 + i1, in);
            __builtin_amdgcn_s_setprio(0);
        } else if (wave < CHAINS<R> + HELPERS_ALL) {
            __builtin_amdgcn_s_setprio(2);
            help_block<R>(lds, wave - CHAINS<R>, blk, es, nbw);
            __builtin_amdgcn_s_setprio(0);
        }
        if (behind >= in) break;                               // uniform: the last block
        if (wave == WAVES - 1) {
            stage_groups(far, lds.cg[blk & 1]);
            if (lane == 0) lds.next[(blk & 1) ^ 1] = 0;
            // What the next block's strips read of U, into the L2: three blocks' rows at its columns, lines of 128 bytes.
            if (far < in) {
                const int far_w = min(in - far, GB);
                for (int h = 0; h < 3 * GB; h += 2 * 64) {
                    float t[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int l = 4 * h + 64 * q + lane, row = min(i1 + (l >> 2), in - 1), c = min(far + (l & 3) * 32, far + far_w - 1);
                        t[q] = U[int64_t(row) * in64 + c];
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) asm volatile("" ::"v"(t[q]));
                }
            }
        }

        // A list for the waves that are free: the next block's corner and parameters; the strips of its columns, which get the errors
        // of the last block and then this one's, sub-block by sub-block; pieces of the last block's update of the columns behind it.
        // On the matrix cores the last pieces are half as wide, or those who end first would wait for a whole one (a piece takes 18 us).  Whole
        // calls, us, none / 4 / 8 / 14 / all pieces halved: 16 rows, 4096 x 4096 1732 / 1672 / 1632 / 1629 / 1635, 3900 x 2048 629 / 574 / 560 / 552 /
        // 550; 32 rows, 8100 x 3300 2208 / 2143 / 2144 / 2154 / 2183 (4 of them are 8 items there).
        const int n_far = blk > 0 && far < in ? in - far : 0, halves = R / RT;
        const int wide = RT == 16 ? max(0, (n_far + ITEM - 1) / ITEM - NARROW) : (n_far + ITEM - 1) / ITEM;
        const int narrow_at = PIECES_AT + wide * halves, n_items = narrow_at + (max(0, n_far - wide * ITEM) + ITEM / 2 - 1) / (ITEM / 2) * halves;
        int* next = &lds.next[blk & 1];
        auto take = [&] {
            int item = 0;
            if (lane == 0) item = atomicAdd(next, 1);
            return __builtin_amdgcn_readfirstlane(item);
        };
        auto posted = [&](int n) {
#pragma unroll
            for (int ch = 0; ch < CHAINS<R>; ++ch) wait_for(&lds.posted[ch], mark(blk, n));
        };
        int item = take();
        while (item < n_items) {
            if (item >= PIECES_AT) {
                if constexpr (RT == 16) {
                    if (item < narrow_at)
                        item = update_behind<R, 2>(Wrows, U, es_last, n_rows, in, int64_t(i1) - GB, far, item - PIECES_AT, narrow_at - PIECES_AT,
                                                   [&] { return take() - PIECES_AT; }) + PIECES_AT;
                    else
                        item = update_behind<R, 1>(Wrows, U, es_last, n_rows, in, int64_t(i1) - GB, far + wide * ITEM, item - narrow_at,
                                                   n_items - narrow_at, [&] { return take() - narrow_at; }) + narrow_at;
                } else {
                    const int piece = item - PIECES_AT;
                    const int rt = R == RT ? 0 : (piece & 1) * RT, cc = R == RT ? piece : piece >> 1;
                    if (rt < n_rows)
                        update_item<R, RT, CPL>(Wrows + rt * in64, U, es_last + rt, n_rows - rt, in, int64_t(i1) - GB, far + cc * (64 * CPL));
                    item = take();
                }
                continue;
            }
            if (item == 0) {
                // This block's corner and parameters at a sub-block have served when the chain is through the next and the helpers with it.
                Stage<R> st[2];
                auto fetch = [&](int b, int sub) {
                    st[b].fetch(U, in, behind, next_w, sub, lds.cg[(blk & 1) ^ 1], row0, n_rows, n_cg, mfmt, st_scales, st_zeros);
                };
                auto put = [&](int b, int sub) {
                    posted(min(sub + 2, GB / SB));
#pragma unroll
                    for (int h = 0; h < HELPERS_ALL; ++h) wait_for(&lds.done[h], mark(blk, sub + 2));
                    st[b].put(lds, sub, mfmt);
                };
                fetch(0, 0);
#pragma unroll 1
                for (int sub = 0; sub < GB / SB; sub += 2) {
                    fetch(1, sub + 1);
                    put(0, sub);
                    if (sub + 2 < GB / SB) fetch(0, sub + 2);
                    put(1, sub + 1);
                }
                item = take();
                continue;
            }
            const int lane = fresh(tid & 63), c = Strip<R>::COLS * (item - 1) + 4 * (lane % Strip<R>::CL);
            const uint32_t pitch = 4u * static_cast<uint32_t>(fresh_uniform(in)), col = 4u * static_cast<uint32_t>(min(c, next_w - 1));
            const int u_row = blk > 0 ? i1 - GB : i1;
            const update::Matrix W(Wrows + behind, int64_t(n_rows) * in - behind), Urows(U + int64_t(u_row) * in64 + behind, (in64 - u_row) * in64 - behind);
            Strip<R> s;
            float u[2][SB][4];
#pragma unroll
            for (int r = 0; r < Strip<R>::RQ; ++r)
                W.load(s.v[r], static_cast<uint32_t>(min(Strip<R>::row(lane, r), n_rows - 1)) * pitch + col, 0);
            uint32_t row = 0;                                  // offset of the row of U to fetch next
            auto fetch = [&](int b) {
#pragma unroll
                for (int kk = 0; kk < SB; ++kk) {
                    Urows.load(u[b][kk], col, row);
                    row += pitch;
                }
            };
            fetch(0);
            if (blk > 0) {
#pragma unroll 1
                for (int k = 0; k < GB; k += 2 * SB) {
                    fetch(1);
                    s.apply(es_last, k, lane, u[0]);
                    fetch(0);                                  // (at the end this block's first)
                    s.apply(es_last, k + SB, lane, u[1]);
                }
            }
#pragma unroll 1
            for (int sub = 0; sub < GB / SB; sub += 2) {
                fetch(1);
                posted(sub + 1);
                s.apply(es, sub * SB, lane, u[0]);
                if (sub + 2 < GB / SB) fetch(0);
                posted(sub + 2);
                s.apply(es, (sub + 1) * SB, lane, u[1]);
            }
            // the chain is through, and the strip with it
#pragma unroll
            for (int r = 0; r < Strip<R>::RQ; ++r)
                *reinterpret_cast<float4*>(&lds.w[Strip<R>::row(lane, r)][c]) = make_float4(s.v[r][0], s.v[r][1], s.v[r][2], s.v[r][3]);
            item = take();
        }
        __syncthreads();
    }
}

// Which form and how many rows per workgroup: the least of the models below, in us without what all forms share (the copies around the
// sweep).  Their constants were fitted to whole calls at 760 sizes (8 to 100000 rows, 16 to 28672 channels) and then moved by a few percent to
// where the choice is best.  At 300 other sizes it is 0.50 % slower than the best form on average (0.17 % from 128 channels on) and 11 % at worst
// there (17590 x 6192); constants from before the step between blocks ran beside the chain took one launch too rarely, 1.13 times
// the present time above 8192 rows.  us, one launch [rows per workgroup] / a launch per block (all of them: profiles/gptq_per_oc_forms.md):
//   one round of workgroups           2048 x 2048  420 [8] / 1098      4096 x 4096  1612 [16] / 2653   8192 x 512  126 [32] / 302
//   rows per workgroup                3072 x 3072  950 [12], 987 [16]  1024 x 4096  697 [4], 1100 [8]  9216 x 1024  531 [24], 580 [32]
//   several rounds                    20000 x 256  157 [32] / 233      28672 x 1024  1162 [32] / 1409  100000 x 256  616 [32] / 801
//   many channels, updates dear       8704 x 8192  15910 [12] / 13220  5632 x 11008  16860 [24] / 15270  9216 x 4096  4571 [12] / 4322
//   few rows and very many channels   8 x 16384  9926 [4] / 8689
//
// In one launch: rounds of workgroups, each of which takes a block's chain and the strips and the update of the columns behind the next
// block, spread over its waves, and at the last block its chain alone.  Beyond 10000 channels a block's rows of U no longer fit an XCD's L2, and
// few workgroups wait for them by themselves.
struct Parts {
    int rows;
    double start, last, block, behind, column;  // of a round; of the last block's chain; of another block; more with columns behind the next; per such column
};
constexpr Parts PARTS[] = {{4, 4.9, 7.8, 11.4, 0.4, 6.0e-3},    {8, 5.4, 8.7, 11.9, 8.8, 8.95e-3},  {12, 6.0, 10.0, 14.8, 7.0, 15.0e-3},
                           {16, 6.3, 10.1, 15.9, 2.9, 18.0e-3}, {24, 7.3, 13.3, 24.5, 0.8, 31.8e-3}, {32, 8.7, 12.8, 26.8, 0.0, 35.7e-3}};

inline double rows_us(const Parts& p, int64_t out, int64_t in) {
    const int64_t wgs = (out + p.rows - 1) / p.rows, last = in - (in - 1) / GB * GB;
    const double column = p.column * (in > 10000 ? 1.0 + 0.54 / std::sqrt(double(wgs)) : 1.0);
    // blocks before the last, and those behind the first with columns (in - 2 GB - GB k of them, k = 1 .. n_far) behind the next block
    const int64_t n = (in - 1) / GB, n_far = in > 2 * GB ? (in - 2 * GB - 1) / GB : 0, far = n_far * (in - 2 * GB) - GB * n_far * (n_far + 1) / 2;
    const double us = p.start + double(n) * p.block + double(n_far) * p.behind + column * double(far) +
                      p.last * double(last / SB * SB) / GB + 0.36 * double(last % SB);
    return us * double((wgs + 255) / 256);
}
inline const Parts& best_parts(int64_t out, int64_t in) {
    const Parts* best = PARTS;
    for (const Parts& p : PARTS)
        if (rows_us(p, out, in) < rows_us(*best, out, in)) best = &p;
    return *best;
}

// A launch per block (gptq_blocks.h): workgroups of 64 rows, in rounds; a short launch for the next block's columns; the rest of
// the update beside the next block's chain, most of the shorter one of the two showing where the chain's workgroups fill the chip.  Channels
// that are no multiple of 16 or of four store codes and errors in smaller pieces.
// (Fitted with the side stream on a hardware queue of its own; where it shares the context's, this form takes up to 1.15 times as
// long: 8704 x 8192 13100 us and 15000.)
inline double blocks_us(int64_t out, int64_t in) {
    const int64_t wgs = (out + 63) / 64;
    const double rounds = double((wgs + 255) / 256), full = std::min(1.0, double(wgs) / 256.0), column = 4.51e-6 * double(out);
    const double block = (49.2 + (in % 4 ? 4.2 : 0.0) + (in % 16 ? 7.6 : 0.0)) * rounds;
    double us = 4.6, bulk = 0.0;
    for (int64_t i1 = 0; i1 < in; i1 += GB) {
        const int64_t w = std::min<int64_t>(in - i1, GB), behind = in - i1 - w;
        const double chain = block * double(w) / GB;
        us += std::max(bulk, chain) + 0.73 * full * std::min(bulk, chain);
        if (behind > 0) us += 20.2 + 0.086e-3 * double(in) + column * double(std::min<int64_t>(behind, GB));
        bulk = column * double(std::max<int64_t>(behind - GB, 0));
    }
    return us;
}

inline int rows_per_group(int64_t out, int64_t in) { return best_parts(out, in).rows; }
// Whether this form is the faster one for [out, in]; else a launch per block.  (Of two alike, the one that needs no second stream.)  Up to 32
// channels all calls are starts and ends of launches, and this form takes 8 to 10 us more at some sizes than at others, for a reason that was not
// found: 2048 x 16 15.8 us and 3072 x 16 24.3, a launch per block 17.7 and 18.9.
inline bool better(int64_t out, int64_t in) {
    if (in <= 32 && out >= 2048) return false;
    return rows_us(best_parts(out, in), out, in) <= 1.03 * blocks_us(out, in);
}

template <int R>
hipError_t allow_lds_of() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(gq_rows<R>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(sizeof(Lds<R>)));
}
inline hipError_t allow_lds() {
    for (const hipError_t e : {allow_lds_of<4>(), allow_lds_of<8>(), allow_lds_of<12>(), allow_lds_of<16>(), allow_lds_of<24>(),
                               allow_lds_of<32>()})
        if (e != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace rows

}  // namespace
