// The per-OC GPTQ sweep in one launch (gfx950).  Included by gptq.hip.
//
// With static groups (per-OC) the rows of W do not depend on each other, so a workgroup can take its R rows through
// every channel without meeting another workgroup.  Eight waves:
//   * wave 0 walks the 128 channels of block b: the chain of rounding decisions, latency bound; with 12 rows and more a
//     second wave takes the block's columns behind the next 16;
//   * meanwhile the others apply the errors of block b - 1 to the columns behind block b (a rounded product and a rounded
//     difference per element and channel, which is the definition's sequence, so no fma); wave 0 joins them when its
//     chain is done;
//   * then all waves apply block b's errors to block b + 1's columns, on their way from memory into LDS.
// Two barriers per block, two counters between the chain's waves, and nothing else to wait for.  The launches per block and the two streams this replaces
// left the chip idle around every short launch.  The whole sweep of a 4096 x 4096 layer, 3 bits: 3.3 ms then, 2.1 ms
// in one launch with products and differences in vector instructions, 1.7 ms with the products behind the block on the
// matrix cores (16 and 32 rows per workgroup) and two waves at the chain; 64 to 1024 rows of that width 0.9 ms (the chain alone).
//
// Rows per workgroup: few enough that the chip's 256 compute units all have a workgroup (16 at 4096 rows), so that
// the update is spread over the whole chip; the chain takes much the same time for 4 rows as for 64.  rows_per_group
// picks R from the sizes.
//
// Registers: with 32 rows 26 vector registers do not fit and live in scratch, with 8 rows 12, otherwise none.  They are values
// that hold over the block loop; none is read inside the sixteen channels' chain or the updates' product loops.
//
// Order of the updates of one element: blocks in order, channels inside a block in order, whichever wave applies
// them; every update is one product and one difference.  Hence the same bits as a plain channel-by-channel loop.
#pragma once

#include "common.h"
#include "fastdiv.h"
#include "gptq_chain.h"
#include "gptq_update.h"
#include "scale_format.h"

#include <type_traits>

namespace {

namespace rows {

using namespace chain_ns;

constexpr int WAVES = 8;
constexpr int SECOND = 4;               // the wave beside wave 0's chain, on the same SIMD

template <int R>
constexpr int pow2_rows() { return R <= 4 ? 4 : R <= 8 ? 8 : R <= 16 ? 16 : 32; }

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
    float ut[GB][PITCH];               // ut[c][k] = U[i1 + k][i1 + c], the block's corner, transposed
    float w[R][PITCH];                 // the block's columns of the rows, as the chain finds them
    float e[2][E_WORDS<R>];            // errors (e_at) of this block and the last
    float2 sc[GB][R];                  // static scale of (channel, row) and its reciprocal (NaN: outside fastdiv's range)
    float rd[GB];                      // 1 / U_ii of the block's channels (NaN likewise)
    int cg[2][GB];                     // static group of the channels of this block and the next
    uint8_t zp[GB][R];                 // static zero-point
    int next;                          // next item of the update behind the block
    int posted, done;                  // sub-blocks whose errors are in `e`; whose errors the second wave has applied
};

// A whole sub-block of 16 channels for one row per lane, everything in registers, with the short quotients
// (gptq_chain.h).  Returns false in a lane whose checks failed: nothing of the result is then to be used.  e: the
// errors; qpk: the codes.
template <int R>
__device__ __forceinline__ bool chain16(const float* wrow, const float* ut, const float* rd, const float2* sc, const uint8_t* zp,
                                        float qmax, float (&e)[SB], uint32_t (&qpk)[SB / 4]) {
    float w[SB], s[SB], y[SB], z[SB];
#pragma unroll
    for (int c = 0; c < SB; c += 4) {
        const float4 t = *reinterpret_cast<const float4*>(wrow + c);
        w[c] = t.x; w[c + 1] = t.y; w[c + 2] = t.z; w[c + 3] = t.w;
    }
#pragma unroll
    for (int c = 0; c < SB; ++c) {
        const float2 t = sc[c * R];
        s[c] = t.x;
        y[c] = t.y;
        z[c] = static_cast<float>(zp[c * R]);
    }
#pragma unroll
    for (int c = 0; c < SB / 4; ++c) qpk[c] = 0u;
    Check check;
    // The corner of U (row cc of `ut` holds U[c][cc] for c <= cc) and the reciprocals of its diagonal, four columns at
    // a time and two channels ahead of their use: all of it at once would not fit the registers.
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
        const float d = ub[c][c];
        // k = code - zero: clamping before or after the zero point is added is the same on integers
        const float quo = w[c] * y[c], near = rintf(quo);
        const float k = __builtin_amdgcn_fmed3f(near, -z[c], qmax - z[c]);
        const float num = w[c] - s[c] * k;
        e[c] = fastdiv(num, d, yd[c]);
#pragma unroll
        for (int cc = 0; cc < SB; ++cc) {
            if (cc > c) {
                const float upd = e[c] * ub[cc][c];
                w[cc] = w[cc] - upd;
            }
        }
        qpk[c / 4] = __builtin_amdgcn_cvt_pk_u8_f32(k + z[c], c & 3, qpk[c / 4]);
        check.code(quo, near);
        check.error(num, d, yd[c], e[c]);
    }
    return check.fine();
}

// The same channel by channel in LDS with plain divisions: the ragged end of a row, and values outside the fast
// quotient's range.  n <= 16 channels; `par(c)` gives channel c's scale and zero-point, `put(c, code)` takes its code.
// Lanes that hold the same row do the same reads and writes in the same instruction.
template <int R, typename Par, typename Put>
__device__ __forceinline__ void chain_slow(float* wrow, const float* ut, float* es_col, int n, float qmax, Par par, Put put) {
#pragma unroll 1
    for (int c = 0; c < n; ++c) {
        float sc, zp;
        par(c, sc, zp);
        const float w = wrow[c];
        float q = rintf(w / sc) + zp;
        q = fminf(fmaxf(q, 0.0f), qmax);
        put(c, static_cast<uint8_t>(q));
        const float e = (w - sc * (q - zp)) / ut[c * PITCH + c];
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
    constexpr int KB = 8;                                      // channels per step: their U entries travel one step ahead
    const int lane = threadIdx.x & 63, in = fresh_uniform(in_);
    uint32_t col[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) col[q] = static_cast<uint32_t>(min(c0 + lane + 64 * q, in - 1));   // past the end: read, never stored
    float v[RT][CPL];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const uint32_t at = static_cast<uint32_t>(min(r, n_rows - 1)) * static_cast<uint32_t>(in);
#pragma unroll
        for (int q = 0; q < CPL; ++q) v[r][q] = Wrows[at + col[q]];
    }
    float u[2][KB][CPL];
    const float* urow = U + k0 * in;                           // the row to fetch next
    auto fetch = [&](int b) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
#pragma unroll
            for (int q = 0; q < CPL; ++q) u[b][kk][q] = urow[col[q]];
            urow += in;
        }
    };
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
    };
    errors(0, 0);
    fetch(0);
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
        fetch(1);
        step(0, k);
        if (k + 2 * KB < GB) fetch(0);
        step(1, k + KB);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int q = 0; q < CPL; ++q)
            if (r < n_rows && c0 + lane + 64 * q < in) Wrows[static_cast<uint32_t>(r) * static_cast<uint32_t>(in) + col[q]] = v[r][q];
    }
}

// The update behind a block for workgroups of 16 and 32 rows, the products on the matrix cores (gptq_update.h): items of 16
// rows x 128 columns from column c_first on, as `next` gives them out.  Two waves per SIMD keep the
// vector pipes busy only if neither waits for memory, so the next item's columns of W, and its first entries of U, are on
// their way while this one is worked on; and an instruction beside the differences costs a wave as much as one of them, so
// two products share a channel's errors and row of U, and four channels a read of the errors (64 columns and a read per
// channel: 12 us per pair of items, 90 us for the 3712 columns of the third block of 4096 x 4096, 16 rows; 83 so).
template <int R>
__device__ __forceinline__ void update_behind(float* __restrict__ Wrows, const float* __restrict__ U, const float* es, int n_rows,
                                              int in_, int64_t k0, int c_first, int* next) {
    constexpr int RT = 16, COLS = 128, KB = 8;                 // KB channels per step: their U entries travel one step ahead
    const int lane = fresh(threadIdx.x & 63), in = fresh_uniform(in_);
    const uint32_t pitch = 4u * static_cast<uint32_t>(in);
    const update::Matrix W(Wrows), Urows(U + k0 * in);
    const int halves = n_rows > RT ? 2 : 1, n_items = (in - c_first + COLS - 1) / COLS * halves;
    auto take = [&] {
        int item = 0;
        if (lane == 0) item = atomicAdd(next, 1);
        return __builtin_amdgcn_readfirstlane(item);
    };
    int item = take();
    if (item >= n_items) return;
    auto row0_of = [&](int item) { return halves == 1 ? 0 : (item & 1) * RT; };
    auto col0_of = [&](int item) { return c_first + (halves == 1 ? item : item >> 1) * COLS; };
    auto u_offset = [&](int item, int q) { return 4u * static_cast<uint32_t>(min(col0_of(item) + 64 * q + lane, in - 1)); };
    auto e_first = [&](int item) { return es + e_at<R>(0, row0_of(item) + (lane & 15)); };
    // past the last row or column: read, never stored
    auto load = [&](int item, update::f32x16 (&v)[2]) {
        const int rt = row0_of(item), c0 = col0_of(item);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t row = static_cast<uint32_t>(min(rt + 4 * (lane >> 4) + r, n_rows - 1)) * pitch;
#pragma unroll
            for (int b = 0; b < 8; ++b)
                v[b >> 2][4 * (b & 3) + r] = W.load(row + 4u * static_cast<uint32_t>(min(c0 + 16 * b + (lane & 15), in - 1)), 0);
        }
    };
    float u[2][KB][2];
    auto fetch = [&](int b, int k, const uint32_t (&col)[2]) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk)
#pragma unroll
            for (int q = 0; q < 2; ++q) u[b][kk][q] = Urows.load(col[q], (k + kk) * pitch);
    };
    update::f32x16 v[2], v_next[2], p[2];
    uint32_t ucol[2] = {u_offset(item, 0), u_offset(item, 1)};
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
        const uint32_t ucol_next[2] = {u_offset(then, 0), u_offset(then, 1)};
        const float* e_next = e_first(then);
        auto steps = [&](int k_begin) {
#pragma unroll 1
            for (int k = k_begin; k < k_begin + GB / 2; k += 2 * KB) {
                const bool last = k + 2 * KB == GB;            // behind the block's last channel come the next item's first
                const float* e_behind = last ? e_next : e_row + k + 2 * KB;
                const uint32_t ucol2[2] = {last ? ucol_next[0] : ucol[0], last ? ucol_next[1] : ucol[1]};
#pragma unroll
                for (int kk = 0; kk < 2 * KB; ++kk) {
                    if (kk == 0) fetch(1, k + KB, ucol);
                    if (kk == KB) fetch(0, (k + 2 * KB) & (GB - 1), ucol2);
                    if ((kk & 3) == 0)
                        ev[((kk >> 2) + 1) & 1] = *reinterpret_cast<const update::f32x4*>(kk + 4 < 2 * KB ? e_row + k + kk + 4 : e_behind);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int nk = kk + q;
                        __builtin_amdgcn_sched_barrier(0);
                        p[q ^ 1] = update::products16x64(ev[(nk >> 2) & 1][nk & 3], u[(nk / KB) & 1][nk % KB][q ^ 1]);
                        __builtin_amdgcn_sched_barrier(0);
                        v[q] = v[q] - p[q];
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
                    for (int b = 0; b < 8; ++b) W.store(v[b >> 2][4 * (b & 3) + r], first, (rt + r) * pitch + 4 * (c0 + 16 * b));
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int b = 0; b < 8; ++b)
                        if (4 * (lane_s >> 4) + r < rows_here && 16 * b + (lane_s & 15) < cols_here)
                            W.store(v[b >> 2][4 * (b & 3) + r], first, (rt + r) * pitch + 4 * (c0 + 16 * b));
            }
        }
        if (!more) break;
        item = then;
        ucol[0] = ucol_next[0];
        ucol[1] = ucol_next[1];
        e_row = e_next;
        v[0] = v_next[0];
        v[1] = v_next[1];
    }
}

// Columns of the next block (starting at c1, nbw of them) into the strip, with the errors of the block at k0 applied.
// Wave w takes columns 16 w .. 16 w + 15, lane groups of 16 take R / 4 rows each.
template <int R>
__device__ __forceinline__ void update_next(const float* __restrict__ Wrows, const float* __restrict__ U, const float* es, int n_rows,
                                            int in_, int64_t k0, int c1, int nbw, Lds<R>& lds) {
    constexpr int RQ = R / 4, KB = 16;
    const int tid = fresh(threadIdx.x), lane = tid & 63, wave = tid >> 6, in = fresh_uniform(in_);
    const int c = 16 * wave + (lane & 15), rq = (lane >> 4) * RQ;
    const uint32_t col = static_cast<uint32_t>(c1 + min(c, nbw - 1));
    float v[RQ], u[2][KB];
    const float* urow = U + k0 * in;
    auto fetch = [&](int b) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            u[b][kk] = urow[col];
            urow += in;
        }
    };
    auto step = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
#pragma unroll
            for (int r = 0; r < RQ; ++r) {
                const float upd = es[e_at<R>(k + kk, rq + r)] * u[b][kk];
                v[r] = v[r] - upd;
            }
            if (kk % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
    fetch(0);
#pragma unroll
    for (int r = 0; r < RQ; ++r)
        v[r] = Wrows[static_cast<uint32_t>(min(rq + r, n_rows - 1)) * static_cast<uint32_t>(in) + col];
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
        fetch(1);
        step(0, k);
        if (k + 2 * KB < GB) fetch(0);
        step(1, k + KB);
    }
#pragma unroll
    for (int r = 0; r < RQ; ++r) lds.w[rq + r][c] = v[r];
}

// The 16 errors e of the sub-block at s0 onto the columns c0, c0 + CL .. of a row of the strip, up to c_end, NC at a time: a
// column's sixteen differences wait for each other.
template <int R, int CL>
__device__ __forceinline__ void apply16(const Lds<R>& lds, float* wrow, const float (&e)[SB], int s0, int c0, int c_end) {
    constexpr int NC = 2;
    for (int c = c0; c < c_end; c += NC * CL) {
        float v[NC], u[NC][SB];
#pragma unroll
        for (int t = 0; t < NC; ++t) {
            const int ct = min(c + t * CL, GB - 1);              // past the block: read, not stored
            v[t] = wrow[ct];
#pragma unroll
            for (int k = 0; k < SB; k += 4) {
                const float4 q = *reinterpret_cast<const float4*>(&lds.ut[ct][s0 + k]);
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
        for (int t = 0; t < NC; ++t)
            if (c + t * CL < c_end) wrow[c + t * CL] = v[t];
    }
}

// One wave tells another of its workgroup how far it is (everything it has put into LDS included), and waits for that.  Every
// wait of gq_rows ends: wave 0 waits only for what the second wave does with errors posted before, and the second wave
// only for wave 0's next sub-block.
__device__ __forceinline__ void tell(int* count, int n) {
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(count, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wait_for(const int* count, int n) {
    while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) < n)
        __builtin_amdgcn_s_sleep(1);
}

template <int R>
__global__ __launch_bounds__(64 * WAVES, 2) void gq_rows(float* __restrict__ Wp, const float* __restrict__ U,
                                                         const int32_t* __restrict__ perm, int64_t out, int64_t in64, int g,
                                                         float qmax, int mfmt, const float* __restrict__ st_scales,
                                                         const uint8_t* __restrict__ st_zeros, uint8_t* __restrict__ Qp) {
    // items of the update: RT rows x 128 columns on the matrix cores where RT is 16, else RT rows x 64 CPL columns (RT x CPL
    // accumulators; few rows take more columns, so that an LDS read of the errors serves as many products)
    constexpr int RR = pow2_rows<R>(), CL = 64 / RR, CPL = R <= 8 ? 4 : 2, RT = R <= 16 ? R : R / 2;
    // Two waves for the chain: with 16 rows a block's chain takes 23 us so and 31 alone.  Few rows have few columns per lane
    // behind a sub-block, and telling and waiting costs more (4 and 8 rows: 2 % of the sweep).
    constexpr bool TWO = R >= 12;
    extern __shared__ __align__(16) char smem[];
    Lds<R>& lds = *reinterpret_cast<Lds<R>*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = int64_t(blockIdx.x) * R;
    const int n_rows = static_cast<int>(min(out - row0, int64_t(R)));        // > 0
    const int in = static_cast<int>(in64), n_cg = in / g;
    float* __restrict__ Wrows = Wp + row0 * in64;

    // static groups of the channels of the block at i1 (into buffer b)
    auto stage_groups = [&](int i1, int b) {
        const int tid = fresh(threadIdx.x);
        if (tid < GB)
            lds.cg[b][tid] = i1 + tid < in ? static_cast<int>(static_cast<uint32_t>(perm[i1 + tid]) / static_cast<uint32_t>(g)) : 0;
    };
    // The block's corner of U (transposed), the reciprocals of its diagonal, and its static parameters (groups in cg[b]):
    // fetched into registers first, put into LDS when the last block's corner is no longer needed.
    // 8 lanes along a row of U (one 128-byte line), 8 rows: two-way bank conflicts at most on the turned writes.
    constexpr int NP = GB * R / (64 * WAVES);                  // parameters per thread
    float cu[8][4], cd, ps[NP], pz[NP];
    auto fetch_block = [&](int i1, int nbw, int b) {
        const int tid = fresh(threadIdx.x), in = fresh_uniform(static_cast<int>(in64));
        const int c4 = (tid & 7) * 4, kr = tid >> 3;           // 64 rows at a time
        const float* corner = U + i1 * in64 + i1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = kr + 64 * h, c = c4 + 32 * cb + j;
                    cu[4 * h + cb][j] = (k < nbw && c < nbw) ? corner[static_cast<uint32_t>(k) * static_cast<uint32_t>(in) + c] : 0.0f;
                }
        cd = tid < nbw ? corner[static_cast<uint32_t>(tid) * (static_cast<uint32_t>(in) + 1u)] : 1.0f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int idx = tid + 64 * WAVES * j, c = idx / R, r = idx % R;
            const int64_t at = (row0 + min(r, n_rows - 1)) * n_cg + lds.cg[b][c];
            if (mfmt) {
                ps[j] = __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(st_scales)[at]));
                pz[j] = 0.0f;
            } else {
                ps[j] = st_scales[at];
                pz[j] = static_cast<float>(st_zeros[at]);
            }
        }
    };
    auto store_block = [&](int i1, int b) {
        const int tid = fresh(threadIdx.x), c4 = (tid & 7) * 4, kr = tid >> 3;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int j = 0; j < 4; ++j) lds.ut[c4 + 32 * cb + j][kr + 64 * h] = cu[4 * h + cb][j];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int idx = tid + 64 * WAVES * j, c = idx / R, r = idx % R;
            float sc = ps[j], zp = pz[j];
            if (mfmt) {                                        // ps holds the group word's bits
                const uint32_t wd = __float_as_uint(sc);
                sc = word_scale(wd, mfmt);
                zp = word_zero(wd, mfmt);
            }
            lds.sc[c][r] = make_float2(sc, fastdiv_ok(sc) ? 1.0f / sc : __builtin_nanf(""));
            lds.zp[c][r] = static_cast<uint8_t>(zp);
        }
        if (tid < GB) lds.rd[tid] = block_reciprocal(cd);
        if (tid == 0) lds.next = lds.posted = lds.done = 0;
        stage_groups(i1 + GB, b ^ 1);
    };

    // first block: its columns straight into the strip
    stage_groups(0, 0);
    __syncthreads();
    {
        const int nbw = min(in, GB);
        for (int idx = tid; idx < R * GB; idx += 64 * WAVES) {
            const int r = idx / GB, c = idx % GB;
            lds.w[r][c] = (c < nbw && r < n_rows) ? Wrows[static_cast<uint32_t>(r) * static_cast<uint32_t>(in) + c] : 0.0f;
        }
        fetch_block(0, nbw, 0);
        store_block(0, 0);
    }
    __syncthreads();

    const int crow = lane & (RR - 1), ccol = lane / RR;        // the chain's lane: row (replicated CL times), column lane
    const bool row_in = crow < R, row_ok = crow < n_rows;
    for (int i1 = 0, blk = 0; i1 < in; i1 += GB, ++blk) {
        const int nbw = min(in - i1, GB), behind = i1 + nbw;
        float* es = lds.e[blk & 1];
        const float* es_last = lds.e[(blk & 1) ^ 1];
        if (wave == 0) {
            // the chain the workgroup waits for: ahead of the updates that share its SIMD
            __builtin_amdgcn_s_setprio(3);
            float* wrow = &lds.w[row_in ? crow : 0][0];
            for (int s0 = 0; s0 < nbw; s0 += SB) {
                const int sbw = min(nbw - s0, SB);
                float e[SB];
                uint32_t qpk[SB / 4];
                const float* ut = &lds.ut[s0][s0];
                const float2* sc = &lds.sc[s0][row_in ? crow : 0];
                const uint8_t* zp = &lds.zp[s0][row_in ? crow : 0];
                uint8_t* q_out = Qp + (row0 + crow) * in64 + i1 + s0;
                bool fine = sbw == SB && reciprocals_ok(&lds.rd[s0]);       // uniform
                if (fine) fine = chain16<R>(wrow + s0, ut, &lds.rd[s0], sc, zp, qmax, e, qpk);
                if (!__any(row_ok && !fine)) {
                    // errors for the later updates (0 in rows past the end), codes in visiting order
#pragma unroll
                    for (int k = 0; k < SB; ++k) e[k] = row_ok ? e[k] : 0.0f;
                    if (row_in && ccol == 0) {
#pragma unroll
                        for (int k = 0; k < SB; ++k) es[e_at<R>(s0 + k, crow)] = e[k];
                    }
                    if (row_ok && ccol == 0) {
                        if ((reinterpret_cast<uintptr_t>(q_out) & 15u) == 0) {
                            *reinterpret_cast<uint4*>(q_out) = make_uint4(qpk[0], qpk[1], qpk[2], qpk[3]);
                        } else {
#pragma unroll
                            for (int c = 0; c < SB; ++c) q_out[c] = static_cast<uint8_t>(qpk[c / 4] >> (8 * (c % 4)));
                        }
                    }
                } else if (row_in) {
                    chain_slow<R>(wrow + s0, ut, es + e_at<R>(s0, crow), sbw, qmax,
                                  [&](int c, float& a, float& b) { a = sc[c * R].x; b = static_cast<float>(zp[c * R]); },
                                  [&](int c, uint8_t q) { if (row_ok && ccol == 0) q_out[c] = q; });
#pragma unroll
                    for (int k = 0; k < SB; ++k) e[k] = k < sbw && row_ok ? es[e_at<R>(s0 + k, crow)] : 0.0f;
                    if (!row_ok)
                        for (int k = 0; k < sbw; ++k) es[e_at<R>(s0 + k, crow)] = 0.0f;
                }
                // The block's columns behind the sub-block (only a whole sub-block has any); TWO: the next sub-block's, which
                // the second wave has brought up to the sub-block before (the columns behind those are its business).
                if (s0 + SB < nbw) {
                    if constexpr (TWO) {
                        tell(&lds.posted, s0 / SB + 1);
                        if (s0 > 0) wait_for(&lds.done, s0 / SB);
                    }
                    if (row_in) apply16<R, CL>(lds, wrow, e, s0, s0 + SB + ccol, TWO ? min(nbw, s0 + 2 * SB) : nbw);
                }
                // these columns of the strip are this wave's alone while the chain runs, and LDS serves a wave's accesses in order
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (TWO && wave == SECOND) {
            // A sub-block's errors onto the columns behind the next one, beside the next one's chain
            __builtin_amdgcn_s_setprio(2);
            float* wrow = &lds.w[row_in ? crow : 0][0];
            for (int s0 = 0; s0 + 2 * SB < nbw; s0 += SB) {
                wait_for(&lds.posted, s0 / SB + 1);
                if (row_in) {
                    float e[SB];
#pragma unroll
                    for (int k = 0; k < SB; ++k) e[k] = es[e_at<R>(s0 + k, crow)];
                    apply16<R, CL>(lds, wrow, e, s0, s0 + 2 * SB + ccol, nbw);
                }
                tell(&lds.done, s0 / SB + 1);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        if (wave == WAVES - 1 && behind < in) {
            // What the step after this block reads first, into the L2: the block's rows of U at the next block's columns,
            // and the next block's corner (128 lines of 512 bytes each).
            const int next_w = min(in - behind, GB);
            for (int r = lane; r < 4 * (GB + next_w); r += 64) {
                const int line = r >> 2, c = min((r & 3) * 32, next_w - 1);
                const float t = U[(i1 + line) * in64 + behind + c];
                asm volatile("" ::"v"(t));
            }
        }
        // errors of the last block onto the columns behind this one, item by item
        if (blk > 0 && behind < in) {
            if constexpr (RT == 16) {
                update_behind<R>(Wrows, U, es_last, n_rows, in, int64_t(i1) - GB, behind, &lds.next);
            } else {
                const int n_items = (in - behind + 64 * CPL - 1) / (64 * CPL) * (R / RT);
                for (;;) {
                    int item = 0;
                    if (lane == 0) item = atomicAdd(&lds.next, 1);
                    item = __builtin_amdgcn_readfirstlane(item);
                    if (item >= n_items) break;
                    const int rt = R == RT ? 0 : (item & 1) * RT, cc = R == RT ? item : item >> 1;
                    if (rt < n_rows)
                        update_item<R, RT, CPL>(Wrows + rt * in64, U, es_last + rt, n_rows - rt, in, int64_t(i1) - GB,
                                                behind + cc * (64 * CPL));
                }
            }
        }
        if (behind >= in) break;                               // uniform: the last block
        const int next_w = min(in - behind, GB), next_b = (blk + 1) & 1;
        fetch_block(behind, next_w, next_b);
        __syncthreads();
        update_next<R>(Wrows, U, es, n_rows, in, i1, behind, next_w, lds);
        store_block(behind, next_b);
        __syncthreads();
    }
}

// Which form and how many rows per workgroup: the least of the models below, whose constants (us) are fitted to whole calls of 1341
// sizes (8 to 152064 rows, 16 to 28672 channels, a quarter of them no multiple of 16; 2 to 4 bits), in launches per block and with every
// number of rows within 1.3 of the best.  What they choose is 0.2 % slower than the best on average (0.1 % from 128 channels on) and
// 9 % at worst, 14 % below 128 channels, where a call is 17 to 60 us.  They compare; neither estimates the call, which holds two
// permuting copies as well.  The lines they draw, us, one launch [rows per workgroup] / a launch per block:
//   rows in one round of workgroups   2048 x 2048  496 [8] / 1103      4096 x 4096  1729 [16] / 2659   8192 x 1024  385 [32] / 613
//   more rows than that               9216 x 512   336 [24] / 295      28672 x 1024  1471 [32] / 1414  100000 x 256  1083 [32] / 809
//   rounds of 32 rows nearly full     6676 x 384   141 [32] / 211      16384 x 2159  2216 [32] / 2652  40000 x 1000  1832 [32] / 2024
//   many channels, updates dear       8704 x 8192  17220 [12] / 13210  5632 x 11008  17650 [24] / 15520  8 x 16384  10030 [4] / 8760
//   rows per workgroup                3072 x 3072  1067 [12], 1102 [16]   50000 x 1280  4129 [24], 3515 [32]   12288 x 6144  12200 [24], 10373 [16]
//
// In one launch: rounds of workgroups, each of which takes, block by block, the longer of its chain and the update of the
// columns behind it, and a step to the next block.  With 16 and 32 rows the update's products are on the matrix cores, with 12 and
// more the chain has two waves.  (few: a workgroup or two alone wait for U by themselves.)
struct Parts {
    int rows;
    double chain, step, column;        // of a block; to the next one; of a block's update per column
};
constexpr Parts PARTS[] = {{4, 10.5, 11.4, 7.1e-3},  {8, 12.0, 14.6, 11.4e-3},  {12, 12.4, 15.6, 16.1e-3},
                           {16, 9.3, 16.7, 18.2e-3}, {24, 18.8, 18.4, 32.6e-3}, {32, 18.2, 19.2, 37.5e-3}};

inline double rows_us(const Parts& p, int64_t out, int64_t in) {
    const int64_t wgs = (out + p.rows - 1) / p.rows;
    const double few = 1.0 + 0.14 / double(wgs);
    double us = 9.3 + 0.265 * p.rows;
    for (int64_t i1 = 0; i1 < in; i1 += GB) {
        const int64_t w = std::min<int64_t>(in - i1, GB), behind = in - i1 - w;
        const double update = i1 > 0 ? few * p.column * double(behind) : 0.0;
        us += std::max(p.chain * double(w) / GB, update) + (behind > 0 ? p.step : 0.0);
    }
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
// long: 8704 x 8192 13100 us and 15000, in one launch 16900; 9216 x 512 295 and 339, 335.)
inline double blocks_us(int64_t out, int64_t in) {
    const int64_t wgs = (out + 63) / 64;
    const double rounds = double((wgs + 255) / 256), full = std::min(1.0, double(wgs) / 256.0), column = 4.54e-6 * double(out);
    const double block = 44.0 + (in % 4 ? 3.6 : 0.0) + (in % 16 ? 6.5 : 0.0);
    double us = 7.0, bulk = 0.0;
    for (int64_t i1 = 0; i1 < in; i1 += GB) {
        const int64_t w = std::min<int64_t>(in - i1, GB), behind = in - i1 - w;
        const double chain = std::max(0.0, block * double(w) / GB - 4.6) * rounds;
        us += std::max(bulk, chain) + 0.645 * full * std::min(bulk, chain);
        if (behind > 0) us += 22.4 + 0.62e-3 * double(in) + column * double(std::min<int64_t>(behind, GB));
        bulk = column * double(std::max<int64_t>(behind - GB, 0));
    }
    return us;
}

inline int rows_per_group(int64_t out, int64_t in) { return best_parts(out, in).rows; }
// Whether this form is the faster one for [out, in]; else a launch per block.
inline bool better(int64_t out, int64_t in) { return rows_us(best_parts(out, in), out, in) <= blocks_us(out, in); }

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
