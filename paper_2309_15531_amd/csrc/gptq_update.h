// The update of the channels behind a block, products on the matrix cores (gfx950).  Included by gptq.hip.
//
// The definition's sequence per element and channel is a rounded product and a rounded difference, so the contraction
// cannot go through a multiply-add.  A matrix instruction of depth one with a zero addend gives the rounded products alone:
// fma(e, u, +0) is RN(e u) for every e and u (subnormals, infinities and NaN included) but for the sign of a zero product, -0
// becoming +0.  That sign decides at most the sign of a zero channel value, and neither codes, parameters nor dW depend on
// the latter.  What it saves is operands: one register each of errors and of U makes 1024 or 2048 products, where the product
// and the difference in vector instructions read an error from LDS for every two to four of them and waited for those
// reads.  The fp32 matrix instruction does not run beside vector instructions: with two waves per SIMD 2048 products alone
// take 64 cycles, the differences alone 72, both 134, or 3.7e13 elements per second; products and differences in vector instructions
// from registers alone 139 (2.2 cycles each; 4.3 with one wave), 3.5e13.  With one wave per SIMD it is 2.3e13 against 1.8e13.
#pragma once

#include "common.h"
#include "gptq_chain.h"

#include <type_traits>

namespace {

namespace update {

using chain_ns::GB;
using chain_ns::PITCH;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x32 __attribute__((ext_vector_type(32)));

// 64 x 32 products of one channel: lane l gives the error of row l and the entry of U of column l % 32.  Register r of lane l
// is row row_of(r, l), column l % 32.
__device__ __forceinline__ f32x32 products64x32(float e, float u) {
    f32x32 zero;
#pragma unroll
    for (int r = 0; r < 32; ++r) zero[r] = 0.0f;
    return __builtin_amdgcn_mfma_f32_32x32x1f32(e, u, zero, 0, 0, 0);
}
// 16 x 64 products: lane l gives the error of row l % 16 and the entry of U of column l.  Register r of lane l is row
// 4 * (l / 16) + r % 4, column 16 * (r / 4) + l % 16.
__device__ __forceinline__ f32x16 products16x64(float e, float u) {
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
    return __builtin_amdgcn_mfma_f32_16x16x1f32(e, u, zero, 0, 0, 0);
}
__device__ __forceinline__ int row_of(int r, int lane) { return 32 * (r >> 4) + 8 * ((r & 15) >> 2) + 4 * (lane >> 5) + (r & 3); }

// A matrix whose element a lane reaches by a wave-uniform offset (of the row) and one of its own (of the column), in bytes: a
// load or store is then one instruction, the row's offset one scalar addition.  (Global addresses cost 64-bit additions, in
// every lane or in scalar registers, and with two waves per SIMD each instruction beside the differences shows.)  The offsets
// must stay below 2^31: 128 rows of up to 46340 floats do.
struct Matrix {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ explicit Matrix(const float* p)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, 0x7fffffff, 0x00020000)) {}
    // with its end: what a load of several floats reads behind it is 0
    __device__ __forceinline__ Matrix(const float* p, int64_t floats)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, static_cast<int>(min(floats, int64_t(0x1fffffff)) * 4), 0x00020000)) {}
    __device__ __forceinline__ float load(uint32_t lane_bytes, uint32_t uniform_bytes) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_bytes, uniform_bytes, 0));
    }
    __device__ __forceinline__ void store(float v, uint32_t lane_bytes, uint32_t uniform_bytes) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, lane_bytes, uniform_bytes, 0);
    }
    template <int N>
    __device__ __forceinline__ void store(const float (&v)[N], uint32_t lane_bytes, uint32_t uniform_bytes) const {
        typedef uint32_t words __attribute__((ext_vector_type(N)));
        words t;
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = __float_as_uint(v[i]);
        if constexpr (N == 4) __builtin_amdgcn_raw_buffer_store_b128(t, rsrc, lane_bytes, uniform_bytes, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(t, rsrc, lane_bytes, uniform_bytes, 0);
    }
    // N consecutive floats, at any multiple of 4 bytes
    template <int N>
    __device__ __forceinline__ void load(float (&v)[N], uint32_t lane_bytes, uint32_t uniform_bytes) const {
        static_assert(N == 2 || N == 4, "");
        if constexpr (N == 4) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_bytes, uniform_bytes, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(t[i]);
        } else {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane_bytes, uniform_bytes, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] = __uint_as_float(t[i]);
        }
    }
};

constexpr int ROWS = 64;               // of a workgroup
constexpr int COLS = 128, COLS_NARROW = 64;

// Wp[r][jj] -= E[r][k] * U[k][jj], k = i1 .. i1 + GB - 1 in order (product, then difference), for the columns [col0, col1).
// The workgroup's errors go to LDS once; a column's entries of U travel KB channels ahead of their use.  The next channel's
// products are issued before this channel's differences, so that a wave does not wait for them.  Three waves per SIMD: two keep
// the pipes busy, the third starts or ends a tile.  11008 rows x 3840 columns: 248 us with vector instructions alone (eight
// rows per thread), 187 so, 145 for the bare loop.
// A wave takes all rows and 32 of the columns; NARROW, for at most 64 columns, 16 of the rows and all columns, as otherwise two or
// three of the four waves would have none (whole sweeps, us, eight rows per thread / a wave all rows / so: 34154 x 148 248 / 256 /
// 242, 57538 x 138 335 / 344 / 324, 12551 x 192 111 / 111 / 104; 12551 x 200, of 72 columns, 128 / 124).
template <bool NARROW>
__global__ __launch_bounds__(256, 3) void gq_trailing(float* __restrict__ Wp, const float* __restrict__ U, const float* __restrict__ Ep,
                                                      int64_t out, int64_t in64, int64_t i1, int64_t col0, int64_t col1) {
    constexpr int KB = 8, NR = NARROW ? 16 : 32;               // NR elements per lane
    using Products = std::conditional_t<NARROW, f32x16, f32x32>;
    __shared__ __align__(16) float es[ROWS][PITCH];            // [row][channel]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int in = static_cast<int>(in64);
    const int64_t r0 = int64_t(blockIdx.y) * ROWS;
    const int n_rows = static_cast<int>(min(out - r0, int64_t(ROWS)));         // > 0
    const uint32_t pitch = 4u * static_cast<uint32_t>(in);                     // bytes (64 rows of up to 46340 channels fit 32 bits)
    const Matrix Wrows(Wp + r0 * in64), Urows(U + i1 * in64);
    const float* __restrict__ Erows = Ep + r0 * in64 + i1;
    const int c_end = static_cast<int>(col1);
    const int c0 = static_cast<int>(col0) + static_cast<int>(blockIdx.x) * (NARROW ? COLS_NARROW : COLS) + (NARROW ? 0 : 32 * wave);
    // past the end: read, never stored
    const uint32_t ucol = 4u * static_cast<uint32_t>(min(c0 + (NARROW ? lane : lane & 31), c_end - 1));
    auto row = [&](int r, int lane) { return NARROW ? 16 * wave + 4 * (lane >> 4) + (r & 3) : row_of(r, lane); };
    auto col = [&](int r, int lane) { return c0 + (NARROW ? 16 * (r >> 2) + (lane & 15) : lane & 31); };

    float u[2][KB];
    auto fetch = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) u[b][kk] = Urows.load(ucol, (k + kk) * pitch);
    };
    fetch(0, 0);
    if ((in & 3) == 0) {                                       // Ep is scratch, 16-byte aligned; i1 is a multiple of GB
#pragma unroll
        for (int q = 0; q < ROWS * GB / 4 / 256; ++q) {
            const int idx = tid + 256 * q, r = idx / (GB / 4), k = idx % (GB / 4) * 4;
            *reinterpret_cast<f32x4*>(&es[r][k]) =
                *reinterpret_cast<const f32x4*>(Erows + static_cast<uint32_t>(min(r, n_rows - 1)) * static_cast<uint32_t>(in) + k);
        }
    } else {
#pragma unroll 8
        for (int q = 0; q < ROWS * GB / 256; ++q) {
            const int idx = tid + 256 * q, r = idx / GB, k = idx % GB;
            es[r][k] = Erows[static_cast<uint32_t>(min(r, n_rows - 1)) * static_cast<uint32_t>(in) + k];
        }
    }
    const uint32_t first = static_cast<uint32_t>(row_of(0, lane)) * pitch + ucol;
    float v[NR];
    if (!NARROW && n_rows == ROWS) {
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = Wrows.load(first, row_of(r, 0) * pitch);
    } else {
#pragma unroll
        for (int r = 0; r < NR; ++r)
            v[r] = Wrows.load(static_cast<uint32_t>(min(row(r, lane), n_rows - 1)) * pitch + 4u * static_cast<uint32_t>(min(col(r, lane), c_end - 1)), 0);
    }
    __syncthreads();
    f32x4 ev[2];
    const float* e_row = es[NARROW ? 16 * wave + (lane & 15) : lane];
    auto errors = [&](int b, int k) { ev[b] = *reinterpret_cast<const f32x4*>(e_row + (k & (GB - 1))); };
    auto error = [&](int kk) {                                 // of channel kk of 16, the group of four being in its buffer
        const f32x4 t = ev[(kk >> 2) & 1];
        return (kk & 3) == 0 ? t.x : (kk & 3) == 1 ? t.y : (kk & 3) == 2 ? t.z : t.w;
    };
    auto products = [&](float e, float u) {
        if constexpr (NARROW) return products16x64(e, u);
        else return products64x32(e, u);
    };
    Products p[2];
    errors(0, 0);
    p[0] = products(error(0), u[0][0]);
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
#pragma unroll
        for (int kk = 0; kk < 2 * KB; ++kk) {
            // (behind the block's last channel the first ones are read again and not used)
            if (kk == 0) fetch(1, k + KB);
            if (kk == KB) fetch(0, (k + 2 * KB) & (GB - 1));
            if ((kk & 3) == 0) errors(((kk >> 2) + 1) & 1, k + kk + 4);
            const int nk = kk + 1;
            __builtin_amdgcn_sched_barrier(0);
            p[nk & 1] = products(error(nk), u[(nk / KB) & 1][nk % KB]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = v[r] - p[kk & 1][r];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (!NARROW && n_rows == ROWS) {
        if (c0 + (lane & 31) >= c_end) return;
#pragma unroll
        for (int r = 0; r < NR; ++r) Wrows.store(v[r], first, row_of(r, 0) * pitch);
    } else {
        int lane_s = lane;                                     // offsets are worked out again, not held over the loop
        asm volatile("" : "+v"(lane_s));
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int rr = row(r, lane_s), c = col(r, lane_s);
            if (rr < n_rows && c < c_end) Wrows.store(v[r], static_cast<uint32_t>(rr) * pitch + 4u * static_cast<uint32_t>(c), 0);
        }
    }
}

}  // namespace update

}  // namespace
