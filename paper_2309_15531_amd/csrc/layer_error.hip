// Reconstruction error of a quantization candidate (Eq. 1 of Sec. 3.3, squared)
// as the quadratic form  L = tr(dW H dW^T) = sum_o dW_o H dW_o^T,  and the
// first-minimum selection over candidates (App. B procedure).
//
// H is symmetric, so with the scaled strictly-lower triangle Hs and the
// diagonal kept apart in fp32,
//     L_o = sum_j H_jj dW_oj^2  +  2 * sum_n ( sum_{k<n} dW'_ok Hs_nk ) dW'_on ,
// dW' = dW * colscale.  The inner sums are a GEMM E = dW' * Hs^T restricted to
// k < n (half the flops of the full product), run on the matrix cores with
// fp16 operands and fp32 accumulation; E is never stored: the epilogue
// multiplies each tile by the matching dW' entries and reduces along n.
// Row partials are combined in a fixed order (no atomics), so results are
// bit-reproducible.
#include "common.h"
#include "mfma_tile.h"
#include "error_dma.h"

#include <algorithm>


namespace {

using namespace mfma;

// dW (fp32 / fp16 / already scaled fp16) -> dW16 = fp16(dW * d) in the scoring layout if needed, and
// diag[o] = sum_j H_jj dW_oj^2 in fp32.  One block per row.
struct SrcBatch {
    const void* dW[edma::MAX_BATCH];
};

// blockIdx.y = candidate; dW16 and diag are laid out [candidate][...].
__global__ __launch_bounds__(256) void error_prologue(SrcBatch src, int dW_dtype, int64_t out, int64_t in,
                                                      const float* __restrict__ hmeta,
                                                      __half* __restrict__ dW16_all, float* __restrict__ diag_all) {
    __shared__ float s_red[256];
    const int64_t o = blockIdx.x;
    const void* __restrict__ dW = src.dW[blockIdx.y];
    __half* __restrict__ dW16 = dW16_all ? dW16_all + int64_t(blockIdx.y) * score_elems(out, in) : nullptr;
    float* __restrict__ diag = diag_all + int64_t(blockIdx.y) * out;
    const float* d = hmeta;
    const float* hd = hmeta + in;
    float sum = 0.0f;
    for (int64_t j0 = int64_t(threadIdx.x) * 8; j0 < in; j0 += 256 * 8) {
        float w[8];
        if (dW_dtype == ADADIM_DW_F32) {
            const float4 a = *reinterpret_cast<const float4*>(static_cast<const float*>(dW) + o * in + j0);
            const float4 b = *reinterpret_cast<const float4*>(static_cast<const float*>(dW) + o * in + j0 + 4);
            w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w; w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
        } else {
            const int64_t at = dW_dtype == ADADIM_DW_F16_SCALED ? score_index(o, j0, out, in) : o * in + j0;
            const uint4 raw = *reinterpret_cast<const uint4*>(static_cast<const __half*>(dW) + at);
            const __half2* h = reinterpret_cast<const __half2*>(&raw);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 f = __half22float2(h[i]);
                w[2 * i] = f.x;
                w[2 * i + 1] = f.y;
            }
        }
        const float4 da = *reinterpret_cast<const float4*>(d + j0), db = *reinterpret_cast<const float4*>(d + j0 + 4);
        const float4 ha = *reinterpret_cast<const float4*>(hd + j0), hb = *reinterpret_cast<const float4*>(hd + j0 + 4);
        const float dd[8] = {da.x, da.y, da.z, da.w, db.x, db.y, db.z, db.w};
        const float hh[8] = {ha.x, ha.y, ha.z, ha.w, hb.x, hb.y, hb.z, hb.w};
        if (dW_dtype == ADADIM_DW_F16_SCALED) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float u = w[i] / dd[i];  // exact: d is a power of two
                sum += hh[i] * (u * u);
            }
        } else {
            uint4 o16;
            __half2* h = reinterpret_cast<__half2*>(&o16);
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += hh[i] * (w[i] * w[i]);
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = __floats2half2_rn(w[2 * i] * dd[2 * i], w[2 * i + 1] * dd[2 * i + 1]);
            *reinterpret_cast<uint4*>(dW16 + score_index(o, j0, out, in)) = o16;
        }
    }
    s_red[threadIdx.x] = sum;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) s_red[threadIdx.x] += s_red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) diag[o] = s_red[0];
}

// The row sums of a wave's 64 columns (from col0) x 64 rows (from row0), accumulators as in the MFMA mapping with Hs as the first operand.
// The entries of dW' they need: rows row0 + 32 j + lane % 32, columns col0 + 32 i + 8 g + 4 (lane / 32) ..+3.
__device__ __forceinline__ void row_entries(const __half* __restrict__ A, int64_t col0, int64_t row0, int64_t out, int64_t in, uint2 (&aw)[2][4][2]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int64_t n0 = col0 + 32 * i + 8 * g + 4 * (lane >> 5);
                aw[i][g][j] = n0 < in ? *reinterpret_cast<const uint2*>(A + score_index(min(row0 + 32 * j + (lane & 31), out - 1), n0, out, in))
                                      : make_uint2(0u, 0u);
            }
}
// With hmeta_diag (column scales, diag H) half the diagonal term as well.
__device__ __forceinline__ void row_sums(const floatx16 (&acc)[2][2], const uint2 (&aw)[2][4][2], int64_t col0, int64_t in,
                                         const float* __restrict__ hmeta_diag, float (&sum)[2]) {
    const int lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int64_t n0 = col0 + 32 * i + 8 * g + 4 * lh;
            if (n0 >= in) continue;                            // in % 8 == 0: the four columns are inside together
            float hq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (hmeta_diag) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // d = 2^e: the bit pattern of 1/d is 0x7F000000 minus that of d
                    const float r = __uint_as_float(0x7F000000u - __float_as_uint(hmeta_diag[n0 + e]));
                    hq[e] = 0.5f * hmeta_diag[in + n0 + e] * r * r;
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float2 a = __half22float2(*reinterpret_cast<const __half2*>(&aw[i][g][j].x));
                const float2 b = __half22float2(*reinterpret_cast<const __half2*>(&aw[i][g][j].y));
                sum[j] += (acc[i][j][4 * g + 0] + hq[0] * a.x) * a.x;
                sum[j] += (acc[i][j][4 * g + 1] + hq[1] * a.y) * a.y;
                sum[j] += (acc[i][j][4 * g + 2] + hq[2] * b.x) * b.x;
                sum[j] += (acc[i][j][4 * g + 3] + hq[3] * b.y) * b.y;
            }
        }
}

constexpr int MID_TILE = 128;

// The tile kernel of middle-sized layers: 128 columns of Hs x 128 rows of dW per workgroup, 64 x 64 per wave, 64 of the contraction per stage
// through 32 KB of LDS, the next stage's operands on their way in registers.  A tile's stages follow one another at the L2's latency (0.8 us
// each with two or three tiles on a compute unit), which is what bounds these layers: contractions are cut into chunks of `cut` column blocks, and
// three workgroups share a compute unit, so that one's barriers and epilogue are another's products.  Row-major rows come in pieces of 128 bytes,
// the DMA kernel's in pieces of 64 (2 x 1720 x 2760 row-major 73 us there and 2 x 1720 x 2752 blocked 52; here 59 and 53).  The rows and candidates
// of a slot are neighbours in the grid, the longest slots first, and each is on the XCD that has it in every slot, so that an XCD reads an eighth of
// dW (dealt without that 1 x 7008 x 2280 takes 88 us instead of 71; slots dealt to XCDs in runs, 2 x 1720 x 2760 in whole contractions 97, not 66).
__global__ __launch_bounds__(256, 3) void error_mid(edma::Batch batch, const __half* __restrict__ Hs, int64_t out, int64_t in,
                                                    const float* __restrict__ hmeta_diag, float* __restrict__ part, int cut, int n_slots, int n_pairs) {
    constexpr int N = MID_TILE * 8 / THREADS;                  // 16-byte pieces of an operand's stage per thread
    __shared__ __align__(16) char sN[MID_TILE * ROW_BYTES], sO[MID_TILE * ROW_BYTES];
    __shared__ float s_rows[4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int id = blockIdx.x, slot = id / n_pairs, nth = id - slot * n_pairs;
    const int pair = nth < (n_pairs & ~7) ? (nth & ~7) | (id & 7) : nth;       // eight consecutive ids are on the eight XCDs
    const int MB = static_cast<int>((out + MID_TILE - 1) / MID_TILE), nb = static_cast<int>((in + MID_TILE - 1) / MID_TILE);
    const int cand = pair / MB;
    int chunk = 0, back = slot;                                // slots: chunk 0 of the column blocks from the last, chunk 1 of those that have one, ...
    for (; back >= nb - cut * chunk; ++chunk) back -= nb - cut * chunk;
    const __half* __restrict__ A = batch.A[cand];
    const int64_t col0 = int64_t(nb - 1 - back) * MID_TILE, row0 = int64_t(pair - cand * MB) * MID_TILE;
    const int k_end = static_cast<int>(min(in, min(col0 + MID_TILE, int64_t(chunk + 1) * cut * MID_TILE)));
    const int s_begin = chunk * cut * (MID_TILE / KT), s_end = (k_end + KT - 1) / KT;
    const int c = tid & 7, r0 = tid >> 3;
    const __half* pn[N];
    const __half* po[N];
#pragma unroll
    for (int p = 0; p < N; ++p) {                              // rows past the end: read again, never used
        pn[p] = Hs + score_index(min(col0 + r0 + 32 * p, in - 1), 0, in, in) + (score_blocked(in) ? (c >> 2) * (256 * 32) + 8 * (c & 3) : 8 * c);
        po[p] = A + score_index(min(row0 + r0 + 32 * p, out - 1), 0, out, in) + (score_blocked(in) ? (c >> 2) * (256 * 32) + 8 * (c & 3) : 8 * c);
    }
    const int64_t step = score_blocked(in) ? KT / 32 * (256 * 32) : KT;
    uint4 rn[N], ro[N];
    auto fetch = [&](int s) {
        const bool have = KT * s + 8 * c < in;                 // in % 8 == 0
#pragma unroll
        for (int p = 0; p < N; ++p) {
            rn[p] = have ? *reinterpret_cast<const uint4*>(pn[p] + s * step) : make_uint4(0, 0, 0, 0);
            ro[p] = have ? *reinterpret_cast<const uint4*>(po[p] + s * step) : make_uint4(0, 0, 0, 0);
        }
    };
    floatx16 acc[2][2] = {};
    fetch(s_begin);
#pragma unroll 1
    for (int s = s_begin; s < s_end; ++s) {
#pragma unroll
        for (int p = 0; p < N; ++p) {
            *reinterpret_cast<uint4*>(sN + lds_off(r0 + 32 * p, c)) = rn[p];
            *reinterpret_cast<uint4*>(sO + lds_off(r0 + 32 * p, c)) = ro[p];
        }
        __syncthreads();
        if (s + 1 < s_end) fetch(s + 1);
        mma_stage<2, 2>(sN, sO, 64 * wm, 64 * wn, lane, acc);
        __syncthreads();
    }
    uint2 aw[2][4][2];
    row_entries(A, col0 + 64 * wm, row0 + 64 * wn, out, in, aw);
    float sum[2] = {0.0f, 0.0f};
    row_sums(acc, aw, col0 + 64 * wm, in, chunk == 0 ? hmeta_diag : nullptr, sum);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float v = sum[j] + __shfl_xor(sum[j], 32, 64);
        if (lane < 32) s_rows[wave][32 * j + lane] = v;
    }
    __syncthreads();
    const int64_t o = row0 + tid;
    if (tid < MID_TILE && o < out)
        part[(int64_t(cand) * n_slots + slot) * out + o] = s_rows[tid >> 6][tid & 63] + s_rows[2 + (tid >> 6)][tid & 63];
}

constexpr int SMALL_TILE = 64;

// The tile kernel of small layers: no LDS, the operands' fragments straight from memory (they sit in the L2), tiles of 64 columns of
// Hs x 64 rows of dW, the contraction dealt to the four waves in pairs of steps (the 64 bytes that a row of the scoring layout has
// together).  The row sums are linear in the products, so each wave takes its own share of the contraction through the epilogue, and
// only row sums meet.  What a small layer pays in the DMA kernel is latency: a ring to fill, eight stages and an epilogue of 256 x 256 per workgroup.
__global__ __launch_bounds__(256) void error_small(edma::Batch batch, const __half* __restrict__ Hs, int64_t out, int64_t in,
                                                   const float* __restrict__ hmeta_diag, float* __restrict__ part) {
    constexpr int T = SMALL_TILE, AHEAD = 4;                   // steps of 16 on their way ahead of their products
    __shared__ float s_rows[4][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int n_slots = gridDim.x, slot = n_slots - 1 - static_cast<int>(blockIdx.x), cand = blockIdx.z;      // the longest first
    const __half* __restrict__ A = batch.A[cand];
    const int64_t col0 = int64_t(slot) * T, row0 = int64_t(blockIdx.y) * T;
    float sum[2] = {0.0f, 0.0f};
    {
        const int pairs = static_cast<int>((min(in, col0 + T) + 31) / 32);
        // rows past the end: read again, never used
        const __half* pn[2];
        const __half* po[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pn[i] = Hs + score_index(min(col0 + 32 * i + l32, in - 1), 8 * lh, in, in);
            po[i] = A + score_index(min(row0 + 32 * i + l32, out - 1), 8 * lh, out, in);
        }
        const bool blocked = score_blocked(in);
        half8 fn[AHEAD][2], fo[AHEAD][2];
        auto fetch = [&](int b, int i_mine) {
            const int s = 2 * (wave + 4 * (i_mine >> 1)) + (i_mine & 1);
            const int64_t at = blocked ? int64_t(s >> 1) * (256 * 32) + (s & 1) * 16 : int64_t(s) * 16;
            const bool have = 16 * s + 8 * lh < in;            // in % 8 == 0
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fn[b][i] = have ? *reinterpret_cast<const half8*>(pn[i] + at) : half8{};
                fo[b][i] = have ? *reinterpret_cast<const half8*>(po[i] + at) : half8{};
            }
        };
        const int mine = 2 * ((pairs - wave + 3) / 4);         // (a half pair behind the end multiplies zeros)
#pragma unroll
        for (int b = 0; b < AHEAD; ++b)
            if (b < mine) fetch(b, b);
        uint2 aw[2][4][2];
        row_entries(A, col0, row0, out, in, aw);
        floatx16 acc[2][2] = {};
        for (int s = 0; s < mine; s += AHEAD) {
#pragma unroll
            for (int b = 0; b < AHEAD; ++b) {
                if (s + b < mine) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fn[b][i], fo[b][j], acc[i][j], 0, 0, 0);
                    if (s + b + AHEAD < mine) fetch(b, s + b + AHEAD);
                }
            }
        }
        row_sums(acc, aw, col0, in, wave == 0 ? hmeta_diag : nullptr, sum);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float v = sum[j] + __shfl_xor(sum[j], 32, 64);
        if (lane < 32) s_rows[wave][32 * j + lane] = v;
    }
    __syncthreads();
    const int t = threadIdx.x;
    const int64_t o = int64_t(blockIdx.y) * T + t;
    if (t < T && o < out) {
        const float v = (s_rows[0][t] + s_rows[1][t]) + (s_rows[2][t] + s_rows[3][t]);
        part[(int64_t(cand) * n_slots + slot) * out + o] = v;
    }
}

// sum over the block's 256 threads, in every thread
__device__ __forceinline__ double finish_total(double v, double* s_red) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
    __syncthreads();                                          // (s_red may be in use from the last total)
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

// loss_rows[o] = diag[o] + 2*sum_slot part[slot,o] (no diag array: the tile kernel has put half
// the diagonal term into its row sums) for 256 rows per block, a per-block total,
// and, in the block that finishes last, loss = sum of the block totals in block order (so the
// result does not depend on which block that is), which goes to loss_all[at.i[candidate]].
// `ticket` must be zero on entry and is zero again on exit.  With `best` given, the block that writes the launch's last loss also takes the
// argmin of sel_losses[0..n_sel) (first minimum, NaN never wins, as select_first_min): one launch
// and one kernel boundary less than a separate selection.
// Few blocks and little data: what counts is the chain of dependent latencies.  A row's slots are loaded sixteen at a
// time, the totals go through lane exchanges, and what blocks hand to each other are relaxed device-scope atomics that
// bypass the caches, ordered by the wait behind them (loads one behind the other, trees of barriers and cache write-backs:
// 9 us at 4 slots, 11 at 16, 45 at 136; now 6 to 9).
struct LossPlaces {
    int32_t i[edma::MAX_BATCH];
};
__global__ __launch_bounds__(256) void error_finish(const float* __restrict__ diag_all,
                                                    const float* __restrict__ part_all, int64_t out, int n_slots,
                                                    float* __restrict__ loss_rows_all, float* __restrict__ loss_all, LossPlaces at,
                                                    double* __restrict__ block_tot_all,
                                                    unsigned int* __restrict__ ticket_all,
                                                    const float* __restrict__ sel_losses, int n_sel,
                                                    int32_t* __restrict__ best) {
    __shared__ double s_red[4];
    __shared__ bool s_last;
    // blockIdx.y = candidate
    const float* __restrict__ diag = diag_all + int64_t(blockIdx.y) * out;
    const float* __restrict__ part = part_all + int64_t(blockIdx.y) * n_slots * out;
    float* __restrict__ loss_rows = loss_rows_all ? loss_rows_all + int64_t(blockIdx.y) * out : nullptr;
    float* __restrict__ loss = loss_all + at.i[blockIdx.y];
    double* __restrict__ block_tot = block_tot_all + int64_t(blockIdx.y) * gridDim.x;
    unsigned int* __restrict__ ticket = ticket_all + blockIdx.y;
    const int64_t o = int64_t(blockIdx.x) * 256 + threadIdx.x;
    double mine = 0.0;
    if (o < out) {
        float off = 0.0f;
#pragma unroll 16
        for (int sl = 0; sl < n_slots; ++sl) off += part[int64_t(sl) * out + o];
        const float l = (diag_all ? diag[o] : 0.0f) + 2.0f * off;
        if (loss_rows) loss_rows[o] = l;
        mine = static_cast<double>(l);
    }
    const double block_total = finish_total(mine, s_red);
    if (threadIdx.x == 0) {
        __hip_atomic_store(block_tot + blockIdx.x, block_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the total has arrived before the ticket counts it
        s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last) return;
    double tot = 0.0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += 256)
        tot += __hip_atomic_load(block_tot + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tot = finish_total(tot, s_red);
    if (threadIdx.x == 0) {
        __hip_atomic_store(loss, static_cast<float>(tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (best) {
            unsigned int* done = ticket_all + 32;             // candidates of this launch whose loss is written
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loss has arrived, likewise
            if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.y - 1) {
                int b = -1;
                float bv = 0.0f;
#pragma unroll 8
                for (int i = 0; i < n_sel; ++i) {
                    const float v = __hip_atomic_load(sel_losses + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (v != v) continue;
                    if (b < 0 || v < bv) {
                        b = i;
                        bv = v;
                    }
                }
                *best = b < 0 ? 0 : b;
                __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

__global__ void fill_zero_f32(float* p, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// host: pinned memory that takes the index as well, or null.
__global__ void select_first_min(const float* __restrict__ losses, int n, int32_t* __restrict__ best, int32_t* host) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int b = -1;
    float bv = 0.0f;
    for (int i = 0; i < n; ++i) {
        const float v = losses[i];
        if (v != v) continue;            // NaN never wins
        if (b < 0 || v < bv) {
            b = i;
            bv = v;
        }
    }
    *best = b < 0 ? 0 : b;
    if (host) *host = b < 0 ? 0 : b;
}

// Scratch of one scoring launch, wherever it lives (the context's growing slots, or the fixed device array of the
// entry point that may not allocate).
struct ErrScratch {
    float* part;             // per candidate [n_slots, out] row partials
    float* diag;             // per candidate [out] diagonal terms (prologue path only)
    double* block_tot;       // per candidate one double per 256 rows
    unsigned int* ticket;    // 64 counters, zero between launches
    const void* zero16;      // at least 256 zero bytes
    __half* dW16;            // per candidate scaled copy of dW (prologue path only)
};

// Slots of column blocks 0 .. NB - 1 cut into chunks of kb 256-k blocks.
int count_slots(int NB, int kb) {
    int n = 0;
    for (int nb = 0; nb < NB; ++nb) n += nb / kb + 1;
    return n;
}

// The finest cut that is considered, which bounds the scratch: whole contractions when these give two workgroups per
// compute unit, else the largest of the chunks NB / 2^i that does.
void error_slots_finest(int nc, int MB, int NB, int& kb, int& n_slots) {
    for (kb = NB;; kb = kb > 2 ? kb / 2 : 1) {
        n_slots = count_slots(NB, kb);
        if (kb == 1 || int64_t(nc) * MB * n_slots >= 512) return;
    }
}

// Contraction chunk of a launch of nc candidates, in 256-k blocks, and the number of (chunk, column block) slots.
// Whole contractions (one workgroup per tile, the cheapest in prologues and epilogues) when they give two workgroups per
// compute unit.  Below that the chip would run one long column block's contraction with most of it idle, or, cut finely,
// pay the fixed costs in several rounds of workgroups: the chunk is the one whose slowest XCD is done first.  An XCD's 32
// compute units take its units of work (4 slots x up to 8 row blocks, dealt in serpentine order as the kernel does); a unit
// costs its longest slot's time, fixed + blocks, and an epilogue of its own where the chunk does not end in the diagonal
// block (or the width rules the in-loop epilogue out), by as many of the compute units as it has row blocks for.  Up to 32
// workgroups take the longest unit's time, more the units' sum, and a round that is not full half its last unit more.  Only
// the ratios 2 : 5 : 4 matter; compared with measured times of all chunks of 38 launches from 1 x 64 x 4096 to
// 2 x 256 x 16384 the choice is 1.1 % slower than the best chunk on average and 10 % at worst.  Against the finest cut:
// 1 x 4096 x 4096 97 -> 75 us, 2 x 1720 x 2760 109 -> 66, 2 x 2048 x 2048 50 -> 33, 1 x 8192 x 1024 34 -> 25,
// 2 x 1024 x 4096 66 -> 48, 1 x 256 x 11008 71 -> 41.  Choosing takes the host up to 1 us at ordinary sizes and 11 us at
// 1 x 64 x 28672, on every call (profiles/scoring_chunks.md; every launch there is this kernel's).  Returns the estimate of the chosen cut (with `estimate` for
// whole contractions too).
int error_slots(int nc, int MB, int NB, int64_t in, bool estimate, int& kb, int& n_slots) {
    constexpr int FIXED = 2, BLOCK = 5, EPILOGUE = 4;
    error_slots_finest(nc, MB, NB, kb, n_slots);
    if (kb == NB && !estimate) return 0;
    const int kb_min = kb, pairs = nc * MB;
    const bool in_loop = score_blocked(in) && in % edma::BT == 0;
    int best = 0;
    for (int k = NB; k >= kb_min; --k) {
        // (beyond 32 blocks only the shortest chunk of each number of chunks, or choosing would take longer than launching)
        if (NB > 32 && k > 1 && (NB + k - 1) / k == (NB + k - 2) / (k - 1)) continue;
        struct { int rows, load, last; } x[8] = {};           // row blocks in all units, their times' sum, the last unit's time
        int unit = 0, slot = 0, longest = 0, top = 0;
        auto deal = [&] {                                     // a group of 4 slots: a unit per 8 row blocks
            for (int p = 0; p < pairs; p += 8, ++unit) {
                const int n = std::min(8, pairs - p);
                auto& to = x[(unit / 8) & 1 ? 7 - unit % 8 : unit % 8];
                to.rows += n;
                to.load += n * longest;
                to.last = longest;
            }
            top = std::max(top, longest);
            longest = 0;
        };
        for (int c = 0; c * k < NB; ++c)
            for (int nb = NB - 1; nb >= c * k; --nb) {
                const bool diag = nb < (c + 1) * k;           // the chunk ends in the diagonal block
                const int cost = FIXED + BLOCK * (diag ? nb + 1 - c * k : k) + (in_loop && diag ? 0 : EPILOGUE);
                longest = std::max(longest, cost);
                if ((++slot & 3) == 0) deal();
            }
        if (slot & 3) deal();
        int worst = 16 * top;
        for (const auto& v : x)
            if (v.rows > 8) worst = std::max(worst, 2 * v.load + (v.rows % 8 ? 8 * v.last : 0));
        if (best == 0 || worst < best) {
            best = worst;
            kb = k;
            n_slots = slot;
        }
    }
    return best;
}

// The launch of a layer's tiles: tile edge, contraction chunk in blocks of that edge, (chunk, column block) slots.
struct ErrPlan {
    int tile, cut, n_slots;
};
constexpr int64_t SMALL_STEPS = 1200, MID_TILES = 2048, MID_WORK = 20000;
// Row partials and diagonal terms of the largest launches of the smaller tiles (one slot; with s slots a launch has 1 / s of the rows).
constexpr size_t SMALL_SCRATCH_BYTES = 2 * size_t(MID_TILE) * MID_TILES * sizeof(float);
static_assert(SMALL_TILE * SMALL_STEPS <= MID_TILE * MID_TILES, "the scratch has room for the tiles of 64");

// 64: up to 1200 steps of 64 columns x 64 rows x 64 of the contraction, and 10 of these in a row, where little but latency is left.  Scoring
// calls of n candidates, us, tiles of 64 / 128 / 256: 2 x 256 x 256 12.7 / 13.5 / 18.9, 2 x 504 x 504 13.4 / 14.7 / 24.0, 2 x 512 x 512
// 13.8 / 14.6 / 20.9; beyond, 1 x 1000 x 1000 14.5 / 14.7 / 25.8, 2 x 4000 x 264 18.2 / 14.9 / 26.3, 2 x 200 x 800 16.7 / 16.1 / 22.2.
// 128: the chunk whose estimate, 5 per round of 256 tiles and 7 per column block that a compute unit has to go through one after the other or
// in all, is the least (of the chunks 1 .. 12, 16 .. of 63 launches, up to 2 x 3000 x 3000, the choice is 3 % slower than the best on average),
// if it is ahead of the DMA kernel's estimate.  The lines between the two are fits to 165 launches, blocked (time = 12.7 + 0.203 x this against
// 9.9 + 0.081 x the DMA kernel's) and row-major (12.8 + 0.229 x against 12.0 + 0.096 x), set 10 and 5 % to the DMA kernel's side: of 172
// launches none with a smaller tile is slower than there, and 12 that stay there would gain more than 5 % (profiles/scoring_tiles.md).
// DMA kernel / 128, blocked: 2 x 1024 x 1024 25.8 / 17.0, 2 x 1536 x 1536 32.5 / 25.5, 1 x 2560 x 2560 50.0 / 41.9, 2 x 5816 x 1056 60.2 / 36.8, but 2 x 8192 x 1024 36.4 / 41.5, 1 x 1024 x 4096 36.7 / 41.9 (tiles of 256 fit, in one round);
// row-major: 2 x 1000 x 1000 34.3 / 17.3, 2 x 1448 x 1448 44.2 / 25.8, 2 x 1720 x 2760 73 / 59, 1 x 7008 x 2280 86 / 71, 1 x 60000 x 504 93.7 / 54.4,
// but 1 x 1000 x 6000 72 / 84.
ErrPlan error_plan(int nc, int64_t out, int64_t in) {
    const int64_t nb64 = (in + SMALL_TILE - 1) / SMALL_TILE;
    if (nc * ((out + SMALL_TILE - 1) / SMALL_TILE) * (nb64 * (nb64 + 1) / 2) <= SMALL_STEPS && nb64 <= 10)
        return {SMALL_TILE, static_cast<int>(nb64), static_cast<int>(nb64)};
    constexpr int BT = edma::BT;
    const int MB = static_cast<int>((out + BT - 1) / BT), NB = static_cast<int>((in + BT - 1) / BT);
    const int64_t nb = (in + MID_TILE - 1) / MID_TILE, pairs = nc * ((out + MID_TILE - 1) / MID_TILE), work = pairs * (nb * (nb + 1) / 2);
    const bool mid = pairs * nb <= MID_TILES && work <= MID_WORK;
    ErrPlan dma = {BT, 0, 0};
    const int64_t dma_cost = error_slots(nc, MB, NB, in, mid, dma.cut, dma.n_slots);
    if (!mid) return dma;
    ErrPlan best = {};
    int64_t best_cost = 0;                                     // x 256
    for (int64_t cut = 1; cut <= nb; ++cut) {
        int64_t n_slots = 0;
        for (int64_t n = nb; n > 0; n -= cut) n_slots += n;
        const int64_t tiles = pairs * n_slots;
        if (tiles > MID_TILES) continue;
        const int64_t cost = 5 * 256 * ((tiles + 255) / 256) + 7 * std::max(work, 256 * cut);
        if (best.tile == 0 || cost < best_cost) {
            best = {MID_TILE, static_cast<int>(cut), static_cast<int>(n_slots)};
            best_cost = cost;
        }
    }
    const bool ahead = score_blocked(in) ? 14 * best_cost < 256 * (5 * dma_cost - 260) : 5 * best_cost < 256 * (2 * dma_cost - 30);
    return ahead ? best : dma;
}

int set_error_attr(adadim_ctx* ctx) {
    static PerDeviceOnce once;
    const hipError_t err = once.run([] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(edma::error_tiles_dma<0>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, edma::SMEM_BYTES);
    });
    if (err != hipSuccess)
        return adadim_fail(ctx, ADADIM_EHIP, "hipFuncSetAttribute(error_tiles): %s", hipGetErrorString(err));
    return ADADIM_OK;
}

// One launch group: nc <= MAX_BATCH candidates dW[0..nc) scored against Hs; losses / n_all are the whole
// call's loss array (n_all for the fused selection, taken when best_dev is given), `at` the candidates' places in it.
int run_error_batch(adadim_ctx* ctx, int nc, const void* const* dW, int dW_dtype, int64_t out, int64_t in,
                    const __half* Hs, const float* hmeta, float* loss_rows, float* losses, const LossPlaces& at,
                    int n_all, int32_t* best_dev, const ErrScratch& sc, const ErrPlan& plan) {
    constexpr int BT = edma::BT;
    const int MB = static_cast<int>((out + BT - 1) / BT), NB = static_cast<int>((in + BT - 1) / BT);
    const int n_slots = plan.n_slots;
    const unsigned fin_blocks = static_cast<unsigned>((out + 255) / 256);
    SrcBatch src;
    edma::Batch batch;
    batch.n = nc;
    for (int c = 0; c < edma::MAX_BATCH; ++c) {
        src.dW[c] = c < nc ? dW[c] : nullptr;
        batch.A[c] = c < nc ? (sc.dW16 ? sc.dW16 + size_t(c) * size_t(score_elems(out, in))
                                       : static_cast<const __half*>(dW[c]))
                            : nullptr;
    }
    // Column-scaled fp16 input is consumed as it is and the tile kernel adds the diagonal term;
    // other inputs go through the prologue, which scales them and takes that term in fp32.
    const bool direct = dW_dtype == ADADIM_DW_F16_SCALED;
    if (!direct) {
        ProfScope prof(ctx, "error_prologue");
        hipLaunchKernelGGL(error_prologue, dim3(static_cast<unsigned>(out), nc), dim3(256), 0, ctx->stream, src,
                           dW_dtype, out, in, hmeta, sc.dW16, sc.diag);
    }
    ADADIM_LAUNCH_CHECK(ctx, "error_prologue");
    if (plan.tile != BT) {
        ProfScope prof(ctx, "error_tiles");
        if (plan.tile == MID_TILE) {
            const int n_pairs = nc * static_cast<int>((out + MID_TILE - 1) / MID_TILE);
            hipLaunchKernelGGL(error_mid, dim3(static_cast<unsigned>(n_slots * n_pairs)), dim3(256), 0, ctx->stream, batch, Hs, out, in,
                               direct ? hmeta : nullptr, sc.part, plan.cut, n_slots, n_pairs);
        } else {
            const dim3 grid(static_cast<unsigned>(n_slots), static_cast<unsigned>((out + SMALL_TILE - 1) / SMALL_TILE), static_cast<unsigned>(nc));
            hipLaunchKernelGGL(error_small, grid, dim3(256), 0, ctx->stream, batch, Hs, out, in, direct ? hmeta : nullptr, sc.part);
        }
    } else {
        ProfScope prof(ctx, "error_tiles");
        // units of 4 slots x 8 (candidate, row block) pairs, 32 workgroups each, dealt to 8 XCDs
        const int n_units = ((n_slots + 3) / 4) * ((nc * MB + 7) / 8);
        const unsigned grid = 8u * static_cast<unsigned>((n_units + 7) / 8) * 32u;
        hipLaunchKernelGGL(edma::error_tiles_dma<0>, dim3(grid), dim3(256), edma::SMEM_BYTES, ctx->stream, batch, Hs,
                           out, in, MB, NB, plan.cut * BT, n_slots, sc.zero16, direct ? hmeta : nullptr, sc.part);
    }
    ADADIM_LAUNCH_CHECK(ctx, "error_tiles");
    {
        ProfScope prof(ctx, "error_finish");
        hipLaunchKernelGGL(error_finish, dim3(fin_blocks, nc), dim3(256), 0, ctx->stream,
                           direct ? static_cast<const float*>(nullptr) : sc.diag, sc.part, out, n_slots, loss_rows,
                           losses, at, sc.block_tot, sc.ticket, losses, n_all, best_dev);
    }
    ADADIM_LAUNCH_CHECK(ctx, "error_finish");
    return ADADIM_OK;
}

}  // namespace

int launch_layer_error(adadim_ctx* ctx, int n, const void* const* dW, int dW_dtype, int64_t out, int64_t in,
                       const __half* Hs, const float* hmeta, float* loss_rows, float* losses, int32_t* best_dev,
                       const int32_t* at) {
    constexpr int BT = edma::BT;
    const int MB = static_cast<int>((out + BT - 1) / BT), NB = static_cast<int>((in + BT - 1) / BT);
    ErrScratch sc{};
    void* zero16 = adadim_workspace(ctx, WS_ZERO, 256);
    if (!zero16) return ADADIM_EHIP;
    sc.zero16 = zero16;
    if (ctx->zero_ready_bytes != ctx->ws_bytes[WS_ZERO]) {
        // a fill kernel rather than a memset node, so that the call stays safe to capture in a graph
        const int64_t nz = static_cast<int64_t>(ctx->ws_bytes[WS_ZERO] / 4);
        hipLaunchKernelGGL(fill_zero_f32, dim3(static_cast<unsigned>((nz + 255) / 256)), dim3(256), 0, ctx->stream,
                           static_cast<float*>(zero16), nz);
        ADADIM_LAUNCH_CHECK(ctx, "fill_zero_f32");
        ctx->zero_ready_bytes = ctx->ws_bytes[WS_ZERO];
    }
    int rc = set_error_attr(ctx);
    if (rc != ADADIM_OK) return rc;
    for (int c0 = 0; c0 < n; c0 += edma::MAX_BATCH) {
        const int nc = n - c0 < edma::MAX_BATCH ? n - c0 : edma::MAX_BATCH;
        int kb = 0, n_slots = 0;
        error_slots_finest(nc, MB, NB, kb, n_slots);
        // scratch: per candidate [n_slots, out] row partials; then per candidate [out] diagonal terms.  Room for the finest cut,
        // so that which calls can be recorded after which does not hang on the chunk that is chosen, and of a size of its own for
        // the smaller tiles, whatever this call takes.
        sc.part = static_cast<float*>(adadim_workspace(
            ctx, WS_ERR_PART, size_t(nc) * size_t(n_slots + 1) * size_t(out) * sizeof(float)));
        float* const small_part = static_cast<float*>(adadim_workspace(ctx, WS_ERR_SMALL, SMALL_SCRATCH_BYTES));
        if (!sc.part || !small_part) return ADADIM_EHIP;
        const ErrPlan plan = error_plan(nc, out, in);
        if (plan.tile != BT) sc.part = small_part;
        sc.diag = sc.part + size_t(nc) * size_t(plan.n_slots) * size_t(out);
        // scratch of the final reduction: per candidate one double per 256 rows; then the tickets
        const unsigned fin_blocks = static_cast<unsigned>((out + 255) / 256);
        const size_t fin_bytes = size_t(edma::MAX_BATCH) * fin_blocks * sizeof(double) + 256;
        const bool fin_fresh = ctx->ws_bytes[WS_ERR_FIN] < fin_bytes;
        sc.block_tot = static_cast<double*>(adadim_workspace(ctx, WS_ERR_FIN, fin_bytes));
        if (!sc.block_tot) return ADADIM_EHIP;
        sc.ticket = reinterpret_cast<unsigned int*>(sc.block_tot + (ctx->ws_bytes[WS_ERR_FIN] - 256) / sizeof(double));
        if (fin_fresh) {
            hipLaunchKernelGGL(fill_zero_f32, dim3(1), dim3(64), 0, ctx->stream, reinterpret_cast<float*>(sc.ticket),
                               int64_t(64));
            ADADIM_LAUNCH_CHECK(ctx, "fill_zero_f32");
        }
        sc.dW16 = nullptr;
        if (dW_dtype != ADADIM_DW_F16_SCALED) {
            sc.dW16 = static_cast<__half*>(
                adadim_workspace(ctx, WS_DW16, size_t(nc) * size_t(score_elems(out, in)) * sizeof(__half)));
            if (!sc.dW16) return ADADIM_EHIP;
        }
        LossPlaces places{};
        for (int c = 0; c < nc; ++c) places.i[c] = at ? at[c0 + c] : c0 + c;
        rc = run_error_batch(ctx, nc, dW + c0, dW_dtype, out, in, Hs, hmeta,
                             loss_rows ? loss_rows + size_t(c0) * size_t(out) : nullptr, losses, places, n,
                             c0 + nc == n ? best_dev : nullptr, sc, plan);
        if (rc != ADADIM_OK) return rc;
    }
    return ADADIM_OK;
}

int launch_select(adadim_ctx* ctx, const float* losses, int n, int32_t* best_dev, int32_t* host) {
    {
        ProfScope prof(ctx, "select_first_min");
        hipLaunchKernelGGL(select_first_min, dim3(1), dim3(64), 0, ctx->stream, losses, n, best_dev, host);
    }
    ADADIM_LAUNCH_CHECK(ctx, "select_first_min");
    return ADADIM_OK;
}

// ---------------------------------------------------------------------------------------------
// The scoring call for callers that cannot allocate (code under graph capture, tight serving loops,
// harnesses that forbid hipMalloc): the scratch of the launch lives in a fixed device array instead
// of the context's growing slots.  Layout of the array: [0, 256) zero page (never written after the
// first clear), [256, 512) the 64 counters of error_finish, [512, 512 + 8*MAX_BATCH*fin_blocks)
// block totals, then the row partials.
namespace {

constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(16) << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;

}  // namespace

static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {

// Device address of `scratch` on each GPU (every GPU holds its own copy of the array at its own address);
// looked up once per device, with that device current.
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

int noalloc_scratch(adadim_ctx* ctx, unsigned char** out_ptr, bool* first_use) {
    int dev = -1;
    ADADIM_HIP_TRY(ctx, hipGetDevice(&dev));
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES)
        return adadim_fail(ctx, ADADIM_EINVAL, "adadim_layer_error_batch_select_noalloc: device index %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    *first_use = false;
    if (!g_scratch_ptr[dev]) {
        unsigned char* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return adadim_fail(ctx, ADADIM_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
        *first_use = true;
    }
    *out_ptr = g_scratch_ptr[dev];
    return ADADIM_OK;
}

}  // namespace

int64_t launch_layer_error_noalloc_bytes(int n, int64_t out, int64_t in) {
    constexpr int BT = edma::BT;
    const int MB = static_cast<int>((out + BT - 1) / BT), NB = static_cast<int>((in + BT - 1) / BT);
    int kb = 0, n_slots = 0;
    error_slots_finest(n, MB, NB, kb, n_slots);
    if (const ErrPlan plan = error_plan(n, out, in); plan.tile != BT) n_slots = plan.n_slots;
    const int64_t fin_blocks = (out + 255) / 256;
    return 512 + int64_t(edma::MAX_BATCH) * fin_blocks * 8 + int64_t(n) * n_slots * out * 4;
}

int launch_layer_error_noalloc(adadim_ctx* ctx, int n, const void* const* dW, int64_t out, int64_t in, const __half* Hs,
                               const float* hmeta, float* loss_rows, float* losses, int32_t* best_dev) {
    const ErrPlan plan = error_plan(n, out, in);
    const int64_t need = launch_layer_error_noalloc_bytes(n, out, in);
    if (need > int64_t(NOALLOC_SCRATCH_BYTES))
        return adadim_fail(ctx, ADADIM_EINVAL,
                           "adadim_layer_error_batch_select_noalloc: %d candidates of [%lld, %lld] need %lld bytes of scratch, "
                           "the fixed array holds %lld", n, (long long)out, (long long)in, (long long)need,
                           (long long)NOALLOC_SCRATCH_BYTES);
    unsigned char* ptr = nullptr;
    bool first_use = false;
    int rc = noalloc_scratch(ctx, &ptr, &first_use);
    if (rc != ADADIM_OK) return rc;
    rc = set_error_attr(ctx);
    if (rc != ADADIM_OK) return rc;
    // The zero page and the counters must be zero on entry.  The array keeps the last call's contents (the
    // counters are left at zero by a launch that ran to its end, but not by one that was abandoned), so the
    // first 512 bytes are cleared on every call, by a fill kernel (a memset node would not be safe to record).
    hipLaunchKernelGGL(fill_zero_f32, dim3(1), dim3(128), 0, ctx->stream, reinterpret_cast<float*>(ptr), int64_t(128));
    ADADIM_LAUNCH_CHECK(ctx, "fill_zero_f32");
    const int64_t fin_blocks = (out + 255) / 256;
    ErrScratch sc{};
    sc.zero16 = ptr;
    sc.ticket = reinterpret_cast<unsigned int*>(ptr + 256);
    sc.block_tot = reinterpret_cast<double*>(ptr + 512);
    sc.part = reinterpret_cast<float*>(ptr + 512 + size_t(edma::MAX_BATCH) * size_t(fin_blocks) * 8);
    sc.diag = nullptr;
    sc.dW16 = nullptr;
    LossPlaces places{};
    for (int c = 0; c < n; ++c) places.i[c] = c;
    return run_error_batch(ctx, n, dW, ADADIM_DW_F16_SCALED, out, in, Hs, hmeta, loss_rows, losses, places, n, best_dev, sc,
                           plan);
}
