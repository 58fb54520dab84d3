// GPTQ in the dimension AdaDim selected (paper Sec. 3.3 "Augmenting RTN and GPTQ", App. A.1,
// App. B `gptq_ada`; GPTQ itself is Frantar et al. 2022).  Two calls:
//
//   adadim_gptq_prepare : dead channels, damping, activation order, and the factor U of the
//                         inverse Hessian (inv(H) = U^T U, U upper triangular, visiting order);
//   adadim_gptq_quantize: the channel-by-channel sweep with error feedback.
//
// Factor.  With J the index reversal, A = J H J, A = L L^T (lower Cholesky), H = V V^T for the
// upper triangular V = J L J, hence U = inv(V) = J inv(L) J: one Cholesky and one triangular
// inverse instead of Cholesky / inverse / Cholesky.  Both run in fp64: on this chip an fp64 fma
// costs what an unpacked fp32 fma costs, and the sweep's rounding decisions then see the same
// U (rounded once to fp32) as an fp64 reference.  Blocked right-looking Cholesky (64-wide
// steps inside 512-wide panels: diagonal block in LDS, everything else products) and a triangular
// inverse, by doubling and panel by panel, in the same launches (factor_plan.h).
//
// Sweep.  Rows (per-OC) or row groups (per-IC) are independent.  Per-OC one launch does it all (gptq_rows.h)
// where that is faster, else a launch per block (gptq_blocks.h; rows::better).  Per-IC a
// workgroup keeps its row group's 128-channel block in LDS and walks the channels alone (gptq_groups.h): quantize channel i,
// e = (w - q)/U_ii, w_j -= e*U_ij for the rest of the block; gptq_update.h and gq_next, or the next block's launch, apply the block's errors to the
// channels behind the block, one channel's error at a time.  Every update is a rounded product
// followed by a rounded difference (no fma), in channel order, which fixes the result bit for
// bit.  Per-OC uses static groups (parameters computed beforehand from the original weight and
// looked up by the channel's original index); per-IC recomputes each (row group, channel)'s
// parameters from the channel's current values when it is visited.
#include "common.h"
#include "factor_plan.h"
#include "gptq_blocks.h"
#include "gptq_groups.h"
#include "gptq_rows.h"
#include "gptq_update.h"
#include "scale_format.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace {

constexpr int NB = FACTOR_NB;     // step of the factorization
constexpr int NBO = FACTOR_NBO;   // its panel: the columns behind are updated 512 at a time
constexpr int GB = 128;           // channels per sweep block

// ------------------------------------------------------------------ prepare: order and matrix
__global__ void gq_diag(const float* __restrict__ H, int64_t n, double* __restrict__ d, uint8_t* __restrict__ dead) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const float h = H[j * n + j];
    const bool dd = h == 0.0f;
    dead[j] = dd ? 1 : 0;
    d[j] = dd ? 1.0 : static_cast<double>(h);
}

// damp = percdamp * mean(d), summed in index order by one thread block (fixed tree)
__global__ __launch_bounds__(256) void gq_damp(const double* __restrict__ d, int64_t n, double percdamp,
                                               double* __restrict__ damp) {
    __shared__ double s[256];
    double acc = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += 256) acc += d[j];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *damp = percdamp * (s[0] / static_cast<double>(n));
}

// perm[rank] = j with rank = number of channels that come before j: larger diagonal first,
// equal diagonals by index (a stable descending sort); identity without act_order
__global__ void gq_rank(const double* __restrict__ d, int64_t n, int act_order, int32_t* __restrict__ perm) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n) return;
    if (!act_order) {
        perm[j] = static_cast<int32_t>(j);
        return;
    }
    const double dj = d[j];
    int64_t rank = 0;
    for (int64_t k = 0; k < n; ++k) {
        const double dk = d[k];
        rank += (dk > dj || (dk == dj && k < j)) ? 1 : 0;
    }
    perm[rank] = static_cast<int32_t>(j);
}

// The same ranks in two steps that use the whole chip: block (x, y) counts, for its 256 channels j,
// the channels of the y-th 256 entries of the diagonal that come before j (staged in LDS) and adds the
// count to rank[j] (integer atomics: any order gives the same sum); then perm[rank[j]] = j.
__global__ void gq_zero_i32(int32_t* __restrict__ p, int64_t n) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}
__global__ __launch_bounds__(256) void gq_rank_count(const double* __restrict__ d, int64_t n, int32_t* __restrict__ rank) {
    constexpr int PIECE = 256;                                // (1024: 64 blocks for 4096 channels, 77 us)
    __shared__ double s[PIECE];
    const int64_t j = int64_t(blockIdx.x) * 256 + threadIdx.x, k0 = int64_t(blockIdx.y) * PIECE;
    for (int e = threadIdx.x; e < PIECE; e += 256) s[e] = k0 + e < n ? d[k0 + e] : -1.0;   // diagonal entries are > 0
    __syncthreads();
    if (j >= n) return;
    const double dj = d[j];
    const int m = static_cast<int>(n - k0 < PIECE ? n - k0 : PIECE);
    int c0 = 0, c1 = 0, c2 = 0, c3 = 0;                       // four counters: the adds do not wait for each other
    int e = 0;
    for (; e + 4 <= m; e += 4) {
        c0 += (s[e] > dj || (s[e] == dj && k0 + e < j)) ? 1 : 0;
        c1 += (s[e + 1] > dj || (s[e + 1] == dj && k0 + e + 1 < j)) ? 1 : 0;
        c2 += (s[e + 2] > dj || (s[e + 2] == dj && k0 + e + 2 < j)) ? 1 : 0;
        c3 += (s[e + 3] > dj || (s[e + 3] == dj && k0 + e + 3 < j)) ? 1 : 0;
    }
    for (; e < m; ++e) c0 += (s[e] > dj || (s[e] == dj && k0 + e < j)) ? 1 : 0;
    atomicAdd(rank + j, (c0 + c1) + (c2 + c3));
}
__global__ void gq_rank_place(const int32_t* __restrict__ rank, int64_t n, int32_t* __restrict__ perm) {
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j < n) perm[rank[j]] = static_cast<int32_t>(j);
}

// A = J (P (H' + damp I) P^T) J in fp64: A[a][b] = H'[perm[n-1-a]][perm[n-1-b]] (+ damp on the diagonal),
// H' = H with dead channels' diagonal set to 1
// One row of A per workgroup: the row of H it comes from goes through LDS (a thread per element reading it from memory
// fetched a 64-byte piece for every four bytes: 100 us for a 4096-wide H).  Dynamic LDS: n floats.  Only the lower triangle
// is ever read (the tiles on the diagonal, which are used whole, included).
__global__ __launch_bounds__(256) void gq_gather(const float* __restrict__ H, int64_t n, const int32_t* __restrict__ perm,
                                                 const double* __restrict__ d, const double* __restrict__ damp,
                                                 double* __restrict__ A) {
    extern __shared__ __align__(16) char gg_smem[];
    float* row = reinterpret_cast<float*>(gg_smem);
    const int64_t a = blockIdx.x, pa = perm[n - 1 - a];
    for (int64_t j = threadIdx.x; j < n; j += 256) row[j] = H[pa * n + j];
    __syncthreads();
    const int64_t end = min(n, (a / NB + 1) * NB);
    for (int64_t b = threadIdx.x; b < end; b += 256) A[a * n + b] = b == a ? d[pa] + *damp : static_cast<double>(row[perm[n - 1 - b]]);
}
// the same without LDS, for rows that do not fit it
__global__ void gq_gather_wide(const float* __restrict__ H, int64_t n, const int32_t* __restrict__ perm,
                               const double* __restrict__ d, const double* __restrict__ damp, double* __restrict__ A) {
    const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= n * n) return;
    const int64_t a = idx / n, b = idx % n;
    const int64_t pa = perm[n - 1 - a], pb = perm[n - 1 - b];
    double v = static_cast<double>(H[pa * n + pb]);
    if (a == b) v = d[pa] + *damp;
    A[idx] = v;
}

// ------------------------------------------------------------------ fp64 tiles on the matrix cores
// v_mfma_f64_16x16x4_f64: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; register r of its
// result is D[4 r + l / 16][l % 16].  The vector and the matrix pipe have the same fp64 peak on this
// chip; the matrix form needs a quarter of the LDS reads per flop and no issue slots for the products.
typedef double double4_t __attribute__((ext_vector_type(4)));
constexpr int GT = FACTOR_NB, GK = 32;           // tile edge, contraction chunk
// (128 x 128 tiles were measured too: one workgroup per compute unit instead of four, and the
// products ran a third slower; the matrix pipe wants the other workgroups' waves to fill its gaps.)

// acc += (acc -= with NEG_A) the product of the chunk in LDS: A(i, k) = As[k][i], B(k, j) = Bs[k][j], k < GK.  256 threads:
// 2 x 2 waves, each TS/2 x TS/2 = MT x MT matrix-core tiles of 16 x 16.
template <int TS, bool NEG_A>
__device__ __forceinline__ void dgemm_chunk(const double (*As)[TS + 4], const double (*Bs)[TS + 4], double4_t (&acc)[TS / 32][TS / 32]) {
    constexpr int MT = TS / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int ks = 0; ks < GK; ks += 4) {
        double a[MT], b[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u) {
            a[u] = As[ks + (lane >> 4)][wm * (TS / 2) + u * 16 + (lane & 15)];
            if constexpr (NEG_A) a[u] = -a[u];
            b[u] = Bs[ks + (lane >> 4)][wn * (TS / 2) + u * 16 + (lane & 15)];
        }
#pragma unroll
        for (int u = 0; u < MT; ++u)
#pragma unroll
            for (int v = 0; v < MT; ++v) acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    }
}

// acc += A B (acc -= A B with NEG_A) for one TS x TS tile and k in [k_lo, k_hi), 256 threads.
//   A(i, k) = A_KC ? Ap[i * lda + k] : Ap[k * lda + i], rows i < m_valid;
//   B(k, j) = B_KC ? Bp[j * ldb + k] : Bp[k * ldb + j], columns j < n_valid;
// everything outside the valid ranges reads as zero.  As, Bs: [GK][TS + 4] doubles each.
template <int TS, bool A_KC, bool B_KC, bool NEG_A = false>
__device__ __forceinline__ void dgemm_tile(const double* __restrict__ Ap, int64_t lda, int m_valid,
                                           const double* __restrict__ Bp, int64_t ldb, int n_valid, int64_t k_lo,
                                           int64_t k_hi, double (*As)[TS + 4], double (*Bs)[TS + 4],
                                           double4_t (&acc)[TS / 32][TS / 32]) {
    constexpr int E = TS / 16;                            // elements per thread and operand
    const int t = threadIdx.x;
    // Loads: 16 consecutive lanes read 16 consecutive doubles (one 128-byte line).  For an operand
    // that is contiguous along k they are the chunk's 16 k of one row (rows t/16 + 16 e); for the
    // other form they are 16 rows or columns of one k (k = t/16, rows or columns t%16 + 16 e).
    const int l16 = t & 15, h16 = t >> 4;
    constexpr int KK = GK / 16;                           // 16-wide pieces of a chunk
    double ra[KK][E], rb[KK][E];
    // the next chunk's operands travel from memory to registers while the matrix cores work on this one
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const int64_t k = k0 + 16 * kk + l16, kr = k0 + 16 * kk + h16;
            if constexpr (A_KC) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int row = h16 + 16 * e;
                    ra[kk][e] = (row < m_valid && k < k_hi) ? Ap[row * lda + k] : 0.0;
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int row = l16 + 16 * e;
                    ra[kk][e] = (kr < k_hi && row < m_valid) ? Ap[kr * lda + row] : 0.0;
                }
            }
            if constexpr (B_KC) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int row = h16 + 16 * e;
                    rb[kk][e] = (row < n_valid && k < k_hi) ? Bp[row * ldb + k] : 0.0;
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int col = l16 + 16 * e;
                    rb[kk][e] = (kr < k_hi && col < n_valid) ? Bp[kr * ldb + col] : 0.0;
                }
            }
        }
    };
    if (k_lo < k_hi) fetch(k_lo);
    for (int64_t k0 = k_lo; k0 < k_hi; k0 += GK) {
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (A_KC) As[16 * kk + l16][h16 + 16 * e] = ra[kk][e];
                else As[16 * kk + h16][l16 + 16 * e] = ra[kk][e];
            }
            if constexpr (B_KC) {
#pragma unroll
                for (int e = 0; e < E; ++e) Bs[16 * kk + l16][h16 + 16 * e] = rb[kk][e];
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) Bs[16 * kk + h16][l16 + 16 * e] = rb[kk][e];
            }
        }
        __syncthreads();
        if (k0 + GK < k_hi) fetch(k0 + GK);
        dgemm_chunk<TS, NEG_A>(As, Bs, acc);
    }
}

// visits the tile's elements this lane holds: f(row in tile, column in tile, value)
template <int TS, typename F>
__device__ __forceinline__ void dgemm_each(const double4_t (&acc)[TS / 32][TS / 32], F f) {
    constexpr int MT = TS / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int v = 0; v < MT; ++v)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(wm * (TS / 2) + u * 16 + 4 * r + (lane >> 4), wn * (TS / 2) + v * 16 + (lane & 15), acc[u][v][r]);
}

// fills the lane's elements of a tile: acc = f(row in tile, column in tile)
template <int TS, typename F>
__device__ __forceinline__ void dgemm_fill(double4_t (&acc)[TS / 32][TS / 32], F f) {
    constexpr int MT = TS / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int v = 0; v < MT; ++v)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[u][v][r] = f(wm * (TS / 2) + u * 16 + 4 * r + (lane >> 4), wn * (TS / 2) + v * 16 + (lane & 15));
}

// ------------------------------------------------------------------ M = inv(L), lower
// inv [[A, 0], [C, B]] = [[inv A, 0], [-inv(B) C inv(A), inv B]].  Diagonal blocks of up to a panel by doubling: with the
// blocks of size s inverted, a level pairs them up: a pair covers rows a0 = base + 2 s pair (A) and a0 + s (B, at
// most s rows at the end) of the `w` rows from `base` on.  Two products, every pair and
// every tile in parallel: T = C inv(A) (inv(A) lower triangular: k starts at the tile's
// first column), then M[B rows, A columns] = -inv(B) T (k ends with the tile's last row).
//
// Panel by panel: the rows below the panel at k0 (w wide) gather R = L X, X = inv(L) of the panels so far, in the part of M that
// their own inverse will take, and a panel's rows become X = -inv(diagonal block) R when their turn comes.  That product
// goes to the lower triangle of A, whose columns left of the panel nobody reads any more (R is read by several workgroups).
// Every product is at most 512 deep and as many tiles wide as there are columns.  (T = C inv(A) in one product when a panel's
// turn comes has tiles up to 3584 deep at 4096, 250 us each.)
//
// These products, and the update behind a panel, are the jobs that the factorization's launches carry (factor_plan.h), a workgroup
// per tile.

// tile `tile` of the launch's jobs (none: past their end)
__device__ __forceinline__ void job_tile(const FactorJobs& jobs, int tile, double* __restrict__ A, double* __restrict__ M,
                                         double* __restrict__ T, float* __restrict__ U, int64_t n, double (*As)[GT + 4], double (*Bs)[GT + 4]) {
    // (the first job's fields are read at once, not when it is known that it is the first)
    int i = 0, kind = jobs.job[0].kind, from = jobs.job[0].from, w = jobs.job[0].w, s = jobs.job[0].s, lo = jobs.job[0].lo, hi = jobs.job[0].hi;
    int64_t k0 = jobs.job[0].k0;
    while (i < jobs.n && tile >= jobs.job[i].tiles) tile -= jobs.job[i++].tiles;
    if (i == jobs.n) return;
    if (i > 0) {
        kind = jobs.job[i].kind;
        from = jobs.job[i].from;
        w = jobs.job[i].w;
        s = jobs.job[i].s;
        lo = jobs.job[i].lo;
        hi = jobs.job[i].hi;
        k0 = jobs.job[i].k0;
    }
    tile += from;
    if (kind == FACTOR_FLIP) {
        // U[a][b] = fp32(inv(L)[n-1-a][n-1-b]): upper triangular, visiting order; columns of X left of the panel are in A, the
        // others in M
        const int64_t r = k0 + tile, a = n - 1 - r;
        for (int64_t b = threadIdx.x; b < n; b += 256) {
            const int64_t c = n - 1 - b;
            U[a * n + b] = c <= r ? static_cast<float>((c < k0 ? A : M)[r * n + c]) : 0.0f;
        }
        return;
    }
    double4_t acc[GT / 32][GT / 32] = {};
    if (kind == FACTOR_T || kind == FACTOR_LEVEL) {
        const int across = s / GT, lg = __ffs(across) - 1;           // a power of two
        const int pair = tile >> (2 * lg), m0 = ((tile >> lg) & (across - 1)) * GT, n0 = (tile & (across - 1)) * GT;
        const int64_t a0 = k0 + 2 * int64_t(pair) * s, b0 = a0 + s;
        const int sb = min(static_cast<int>(k0 + w - b0), s);     // > 0 for every pair
        if (m0 >= sb) return;
        const int m_valid = min(sb - m0, GT);
        double* Tp = T + int64_t(pair) * s * s;
        if (kind == FACTOR_T) {
            dgemm_tile<GT, false, false>(M + a0 * n + b0 + m0, n, m_valid, M + a0 * n + a0 + n0, n, GT, n0, s, As, Bs, acc);
            dgemm_each<GT>(acc, [&](int i, int j, double v) {
                if (i < m_valid) Tp[int64_t(m0 + i) * s + n0 + j] = v;
            });
        } else {
            dgemm_tile<GT, true, false>(M + (b0 + m0) * n + b0, n, m_valid, Tp + n0, s, GT, 0, min(sb, m0 + GT), As, Bs, acc);
            dgemm_each<GT>(acc, [&](int i, int j, double v) {
                if (i < m_valid) M[(b0 + m0 + i) * n + a0 + n0 + j] = -v;
            });
        }
    } else if (kind == FACTOR_ROWS) {
        // X's rows of the panel at k0 (w of them), columns left of it
        const int cols = static_cast<int>(k0 / GT), m0 = tile / cols * GT, m_valid = min(w - m0, GT), end = min(hi, m0 + m_valid);
        const int64_t c0 = int64_t(tile % cols) * GT;
        if (lo > 0) dgemm_fill<GT>(acc, [&](int i, int j) { return i < m_valid ? A[(k0 + m0 + i) * n + c0 + j] : 0.0; });
        dgemm_tile<GT, true, false, true>(M + (k0 + m0) * n + k0, n, m_valid, M + k0 * n + c0, n, GT, lo, end, As, Bs, acc);
        dgemm_each<GT>(acc, [&](int i, int j, double v) {
            if (i < m_valid) A[(k0 + m0 + i) * n + c0 + j] = v;
        });
    } else if (kind == FACTOR_SPREAD) {
        // R's rows from k0 + w on, columns 0 .. k0 + w (a multiple of 64)
        const int64_t k1 = k0 + w;
        const int cols = static_cast<int>(k1 / GT);
        const int64_t r0 = k1 + int64_t(tile / cols) * GT, c0 = int64_t(tile % cols) * GT;
        const int m_valid = static_cast<int>(n - r0 < GT ? n - r0 : GT);
        const bool own = c0 >= k0;                            // columns of the panel itself, which nothing was added to yet
        const int first = own ? static_cast<int>(c0 - k0) : 0, begin = max(lo, first);
        if (begin >= hi) return;
        if (!own || begin > first) dgemm_fill<GT>(acc, [&](int i, int j) { return i < m_valid ? M[(r0 + i) * n + c0 + j] : 0.0; });
        dgemm_tile<GT, false, false>(M + k0 * n + r0, n, m_valid, (own ? M : A) + k0 * n + c0, n, GT, begin, hi, As, Bs, acc);
        dgemm_each<GT>(acc, [&](int i, int j, double v) {
            if (i < m_valid) M[(r0 + i) * n + c0 + j] = v;
        });
    } else {
        // A -= L L^T: the tiles of the next panel's columns (`s` of them, those above the diagonal included), or those behind
        const int64_t k1 = k0 + NBO;
        int rt, ct;
        if (kind == FACTOR_NEXT) {
            rt = tile / s;
            ct = tile % s;
            if (ct > rt) return;
        } else {
            factor_behind(tile, rt, ct);
        }
        const int64_t r0 = k1 + int64_t(rt) * GT, c0 = k1 + int64_t(ct) * GT;
        const int m_valid = static_cast<int>(n - r0 < GT ? n - r0 : GT), n_valid = static_cast<int>(n - c0 < GT ? n - c0 : GT);
        dgemm_fill<GT>(acc, [&](int i, int j) { return (i < m_valid && j < n_valid) ? A[(r0 + i) * n + c0 + j] : 0.0; });
        dgemm_tile<GT, false, false, true>(M + k0 * n + r0, n, m_valid, M + k0 * n + c0, n, n_valid, lo, hi, As, Bs, acc);
        dgemm_each<GT>(acc, [&](int i, int j, double v) {
            if (i < m_valid && c0 + j <= r0 + i) A[(r0 + i) * n + c0 + j] = v;
        });
    }
}
// jobs that no step is left to carry
__global__ __launch_bounds__(256, 4) void factor_jobs(double* __restrict__ A, double* __restrict__ M, double* __restrict__ T,
                                                      float* __restrict__ U, int64_t n, FactorJobs jobs) {
    __shared__ double As[GK][GT + 4], Bs[GK][GT + 4];
    job_tile(jobs, static_cast<int>(blockIdx.x), A, M, T, U, n, As, Bs);
}

// ------------------------------------------------------------------ Cholesky, lower, in place
// Diagonal block of width w <= NB = 64, factored and inverted by one workgroup of four waves, blocked by 16.  The whole
// factorization waits for it, so what counts is the length of its dependency chain, not its flops:
//  * A 16 x 16 block on the diagonal is eliminated by wave 0, each of its 16-lane rows doing the same: lane r holds row r of
//    the block and column r of the inverse that grows beside it (16 doubles each).  The chain runs through the pivots
//    alone: pivot c + 1 = q - x^2 / pivot c, q and x being row c + 1's entries of columns c + 1 and c, so that a reciprocal
//    and one fma lie between two of them.  Column c's entries reach the other lanes by a broadcast within the lane row,
//    one instruction each (reads into scalar registers, with the inverse solved afterwards: 43000 cycles for a
//    64-wide block against 23300), and serve the block and the inverse.  The pivots' reciprocal roots scale the inverse's rows at
//    the end; L's own diagonal blocks are not needed.
//  * The rows below are a product with that inverse and the columns behind get their rank-16 update, on the fp64 matrix
//    cores.  Wave 0 takes the next diagonal block alone and goes on to eliminate it; meanwhile the other waves update the
//    other blocks and make row p of the inverse's blocks, -inv(L_pp) sum_k L_pk inv(L)_kq.
// inv(L) goes to the diagonal block of M: it turns the panel's triangular solve into a product and is
// the first level of the triangular inverse.

// lane J's value of every 16-lane row, in all of the row's lanes (data-parallel primitive row_newbcast)
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(__double_as_longlong(v), 0x150 + J, 0xf, 0xf, false));
}
template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}
// LDS writes of this wave before, its LDS reads after: a wave's LDS accesses are served in order
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of the diagonal block's factorization: 39 KB.  inv(L) grows in the block that holds L, so that the launches that end in it
// have four workgroups' LDS on a compute unit (registers allow three).
struct DiagLds {
    static constexpr int LD = NB + 1;
    double t[NB][LD];                                         // 16 x 16 blocks: L below the diagonal, inv(L) on it, inv(L)^T above
    double s[3][16][17];                                      // sum_k L_pk inv(L)_kq of a wave's block
};
// lds.t holds the block (identity padding behind w), visible to the whole workgroup.  Only inv(L) leaves the workgroup:
// nothing reads the diagonal block of L afterwards.
__device__ __forceinline__ void diag_factor(double* __restrict__ M, int64_t n, int64_t k0, int w, DiagLds& lds) {
    constexpr int P = 16, NP = NB / P;
    constexpr auto seq = std::make_integer_sequence<int, P>{};
    auto& t = lds.t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, h16 = lane >> 4;
    // one workgroup that the whole factorization waits for: ahead of the jobs that may share its SIMDs
    __builtin_amdgcn_s_setprio(3);
    // block (ti, tj) -= L_ti,p L_tj,p^T
    auto update = [&](int ti, int tj, int p) {
        double4_t acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = t[P * ti + 4 * r + h16][P * tj + l16];
#pragma unroll
        for (int kk = 0; kk < P; kk += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-t[P * ti + l16][P * p + kk + h16], t[P * tj + l16][P * p + kk + h16], acc,
                                                       0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) t[P * ti + 4 * r + h16][P * tj + l16] = acc[r];
    };
    // block (p, q) of inv(L), q < p, into its place above the diagonal; s: the wave's own
    auto inverse = [&](int p, int q, double (*s)[17]) {
        double4_t acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = q; k < p; ++k)
#pragma unroll
            for (int kk = 0; kk < P; kk += 4) {
                const double b = k == q ? t[P * q + kk + h16][P * q + l16] : t[P * q + l16][P * k + kk + h16];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t[P * p + l16][P * k + kk + h16], b, acc, 0, 0, 0);
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) s[4 * r + h16][l16] = acc[r];
        wave_lds_sync();
        acc = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < P; kk += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-t[P * p + l16][P * p + kk + h16], s[kk + h16][l16], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) t[P * q + l16][P * p + 4 * r + h16] = acc[r];
        wave_lds_sync();
    };
    for (int p = 0; p < NP; ++p) {
        if (wave == 0) {
            if (p > 0) {
                update(p, p, p - 1);
                wave_lds_sync();
            }
            double x[P], y[P];                                // row l16 of the block, column l16 of the inverse
#pragma unroll
            for (int j = 0; j < P; ++j) {
                x[j] = t[P * p + l16][P * p + j];
                y[j] = j == l16 ? 1.0 : 0.0;
            }
            double piv = row_bcast<0>(x[0]), my_piv = 1.0;    // my_piv: pivot l16
            static_for(seq, [&](auto C) {
                constexpr int c = C;
                my_piv = l16 == c ? piv : my_piv;
                double rp = __builtin_amdgcn_rcp(piv);
                rp = fma(fma(-piv, rp, 1.0), rp, rp);
                rp = fma(fma(-piv, rp, 1.0), rp, rp);
                if constexpr (c + 1 < P) {
                    const double xn = row_bcast<c + 1>(x[c]);
                    piv = fma(-(xn * xn), rp, row_bcast<c + 1>(x[c + 1]));
                }
                const double m = x[c] * rp, yc = y[c] * rp;
                static_for(seq, [&](auto J) {
                    constexpr int j = J;
                    if constexpr (j > c) {
                        const double b = row_bcast<j>(x[c]);
                        x[j] = fma(-m, b, x[j]);
                        y[j] = fma(-b, yc, y[j]);
                        asm volatile("" : "+v"(y[j]));        // here and now: put off to the stores, it needs every b held
                    }
                });
            });
            double inv = __builtin_amdgcn_rsq(my_piv);
            inv = inv * fma(-0.5 * my_piv * inv, inv, 1.5);
            inv = inv * fma(-0.5 * my_piv * inv, inv, 1.5);
            // from a pivot that is not positive on, everything is NaN
            const unsigned long long bad = __ballot(!(my_piv > 0.0));
            if (bad && l16 >= __ffsll(bad) - 1) inv = __builtin_nan("");
            static_for(seq, [&](auto J) {
                constexpr int j = J;
                const double v = y[j] * row_bcast<j>(inv);
                if (lane < P) t[P * p + j][P * p + lane] = v;
            });
        } else {
            // beside the elimination: the other blocks' update by column block p - 1, and row p - 1 of the inverse
            int idx = 0;
            for (int ti = p + 1; p > 0 && ti < NP; ++ti)
                for (int tj = p; tj <= ti; ++tj, ++idx)
                    if (idx % 3 == wave - 1) update(ti, tj, p - 1);
            for (int q = 0; q < p - 1; ++q)
                if (q == wave - 1) inverse(p - 1, q, lds.s[wave - 1]);
        }
        __syncthreads();
        // the rows below: L_ti,p = A_ti,p inv(L_pp)^T, a block per wave
        const int ti = p + 1 + wave;
        if (ti < NP) {
            double4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < P; kk += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t[P * ti + l16][P * p + kk + h16], t[P * p + l16][P * p + kk + h16], acc,
                                                           0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) t[P * ti + 4 * r + h16][P * p + l16] = acc[r];
        }
        __syncthreads();
    }
    if (wave < NP - 1) inverse(NP - 1, wave, lds.s[wave]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NB * NB / 256; ++i) {
        const int r = i * (256 / NB) + wave, c = lane, br = r / P, bc = c / P;
        const double v = br == bc ? t[r][c] : (br > bc ? t[c][r] : 0.0);
        if (r < w && c < w) M[(k0 + r) * n + k0 + c] = v;
    }
}

// the first block
__global__ __launch_bounds__(256, 3) void chol_diag_inv(const double* __restrict__ A, double* __restrict__ M, int64_t n, int64_t k0,
                                                        int w) {
    __shared__ DiagLds lds;
    for (int e = threadIdx.x; e < NB * NB; e += 256) {
        const int r = e / NB, c = e % NB;
        lds.t[r][c] = (r < w && c < w) ? A[(k0 + r) * n + k0 + c] : (r == c ? 1.0 : 0.0);   // identity padding
    }
    __syncthreads();
    diag_factor(M, n, k0, w, lds);
}

// L's blocks below the diagonal are kept transposed in the upper triangle of M, whose lower triangle takes inv(L): column c
// of L is M[c][c + 1 ..].  A's own entries there stay as the updates left them, so that several workgroups can each make
// the L they need from them.

// rows below the diagonal block: L21^T = inv(L11) A21^T, 64 rows per block
__global__ __launch_bounds__(256, 4) void chol_panel(const double* __restrict__ A, double* __restrict__ M, int64_t n, int64_t k0,
                                                     int w) {
    __shared__ double As[GK][GT + 4], Bs[GK][GT + 4];
    const int64_t r0 = k0 + w + int64_t(blockIdx.x) * GT;
    const int m_valid = static_cast<int>(n - r0 < GT ? n - r0 : GT);
    double4_t acc[2][2] = {};
    dgemm_tile<GT, true, true>(M + k0 * n + k0, n, w, A + r0 * n + k0, n, m_valid, 0, w, As, Bs, acc);
    dgemm_each<GT>(acc, [&](int c, int i, double v) {
        if (c < w && i < m_valid) M[(k0 + c) * n + r0 + i] = v;
    });
}

// The end of an update's tile: the workgroup of the first tile (the diagonal block at k1, final once this update has
// reached it) goes on to factor and invert that block, without a launch and under the other tiles' products; the others
// store theirs.
__device__ __forceinline__ void chol_tile_end(double4_t (&acc)[GT / 32][GT / 32], double* __restrict__ A, double* __restrict__ M,
                                              int64_t n, int64_t k1, int64_t r0, int64_t c0, int m_valid, int n_valid, DiagLds& lds) {
    if (blockIdx.x == 0 && blockIdx.y == 0) {                 // whole workgroup
        __syncthreads();                                      // the staging buffers are free
        dgemm_each<GT>(acc, [&](int i, int j, double v) { lds.t[i][j] = (i < m_valid && j < n_valid) ? v : (i == j ? 1.0 : 0.0); });
        __syncthreads();
        diag_factor(M, n, k1, m_valid, lds);
    } else {
        dgemm_each<GT>(acc, [&](int i, int j, double v) {
            if (i < m_valid && c0 + j <= r0 + i) A[(r0 + i) * n + c0 + j] = v;
        });
    }
}
// LDS of the two kernels that call it: the product's staging buffers and the factorization's share their space
constexpr size_t STEP_LDS = std::max(sizeof(DiagLds), 2 * GK * (GT + 4) * sizeof(double));

// The update A -= L[., k0 .. k0+w) L[., k0 .. k0+w)^T of the next panel's columns, from k1 on (of everything, where there is no panel
// behind that), with the next diagonal block's factorization.  gridDim.x x rows tiles, then jobs.
__global__ __launch_bounds__(256, 3) void chol_syrk_diag(double* __restrict__ A, double* __restrict__ M, double* __restrict__ T,
                                                         float* __restrict__ U, int64_t n, int64_t k0, int w, int64_t k1, int rows,
                                                         FactorJobs jobs) {
    __shared__ __align__(16) char smem[STEP_LDS];
    double(*As)[GT + 4] = reinterpret_cast<double(*)[GT + 4]>(smem);
    double(*Bs)[GT + 4] = As + GK;
    const int ct = static_cast<int>(blockIdx.x), rt = static_cast<int>(blockIdx.y);
    if (rt >= rows) {
        job_tile(jobs, (rt - rows) * static_cast<int>(gridDim.x) + ct, A, M, T, U, n, As, Bs);
        return;
    }
    if (ct > rt) return;
    __builtin_amdgcn_s_setprio(3);                            // a link of the chain: ahead of the jobs on a shared SIMD
    const int64_t r0 = k1 + int64_t(rt) * GT, c0 = k1 + int64_t(ct) * GT;
    const int m_valid = static_cast<int>(n - r0 < GT ? n - r0 : GT), n_valid = static_cast<int>(n - c0 < GT ? n - c0 : GT);
    double4_t acc[GT / 32][GT / 32];
    dgemm_fill<GT>(acc, [&](int i, int j) { return (i < m_valid && j < n_valid) ? A[(r0 + i) * n + c0 + j] : 0.0; });
    dgemm_tile<GT, false, false, true>(M + k0 * n + r0, n, m_valid, M + k0 * n + c0, n, n_valid, 0, w, As, Bs, acc);
    chol_tile_end(acc, A, M, n, k1, r0, c0, m_valid, n_valid, *reinterpret_cast<DiagLds*>(smem));
}

// One 64-wide step inside a panel: the rows below the diagonal block at k0 and the update of the panel's columns behind it, in one
// launch; gridDim.x x rows tiles, then jobs.  The factorization waits for every step in turn (they leave the chip nearly idle),
// so each workgroup makes the 64 x 64 blocks of L that its tile needs by itself, at two products more, instead of waiting
// for a launch that makes each once (a step of the 4096-wide factor: 34 us in two launches, 28 in one,
// and 22 with the diagonal block's faster elimination).  The first tile
// column's workgroups keep L.
__global__ __launch_bounds__(256, 3) void chol_step(double* __restrict__ A, double* __restrict__ M, double* __restrict__ T,
                                                    float* __restrict__ U, int64_t n, int64_t k0, int rows, FactorJobs jobs) {
    __shared__ __align__(16) char smem[STEP_LDS];
    double(*As)[GT + 4] = reinterpret_cast<double(*)[GT + 4]>(smem);
    double(*Bs)[GT + 4] = As + GK;
    const int ct = static_cast<int>(blockIdx.x), rt = static_cast<int>(blockIdx.y);
    if (rt >= rows) {
        job_tile(jobs, (rt - rows) * static_cast<int>(gridDim.x) + ct, A, M, T, U, n, As, Bs);
        return;
    }
    if (ct > rt) return;
    __builtin_amdgcn_s_setprio(3);
    const int64_t k1 = k0 + NB, r0 = k1 + int64_t(rt) * GT, c0 = k1 + int64_t(ct) * GT;
    const int m_valid = static_cast<int>(n - r0 < GT ? n - r0 : GT), n_valid = static_cast<int>(n - c0 < GT ? n - c0 : GT);
    const bool square = ct == rt;
    double4_t ly[2][2] = {}, lx[2][2] = {}, acc[2][2];        // L^T's blocks of the tile's rows and columns; the tile
    if (!square) dgemm_tile<GT, true, true>(M + k0 * n + k0, n, NB, A + c0 * n + k0, n, n_valid, 0, NB, As, Bs, lx);
    dgemm_tile<GT, true, true>(M + k0 * n + k0, n, NB, A + r0 * n + k0, n, m_valid, 0, NB, As, Bs, ly);
    dgemm_fill<GT>(acc, [&](int i, int j) { return (i < m_valid && j < n_valid) ? A[(r0 + i) * n + c0 + j] : 0.0; });
    if (ct == 0)
        dgemm_each<GT>(ly, [&](int c, int i, double v) {
            if (i < m_valid) M[(k0 + c) * n + r0 + i] = v;
        });
    static_assert(NB == 2 * GK && GT == NB, "a wave row's blocks are one chunk");
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
        if (static_cast<int>(threadIdx.x >> 7) == h) {        // the waves that hold columns GK h .. of L
            dgemm_each<GT>(ly, [&](int c, int i, double v) { As[c - GK * h][i] = v; });
            if (!square) dgemm_each<GT>(lx, [&](int c, int i, double v) { Bs[c - GK * h][i] = v; });
        }
        __syncthreads();
        dgemm_chunk<GT, true>(As, square ? As : Bs, acc);
    }
    chol_tile_end(acc, A, M, n, k1, r0, c0, m_valid, n_valid, *reinterpret_cast<DiagLds*>(smem));
}

// ------------------------------------------------------------------ sweep
// Wp[r][i] = W[r][perm[i]] as fp32, zero for dead channels.  nr rows per workgroup: the rows are read once, in order,
// into LDS (dead channels as zero) and permuted from there (a thread per element reading W[r][perm[i]] from memory
// fetched a separate 64-byte piece for every two bytes it used).  Dynamic LDS: nr * in halves.
// VEC: in % 8 == 0 and 16-byte aligned W and perm, 8-byte aligned dead: 8 channels per load, 4 per store, and a piece of
// perm serves the nr rows.  11008 x 4096, 270 MB: 53 us, where an element at a time takes 68 (11008 x 4090; with a row
// per workgroup 88; 25600 x 2047 70 and 140; 76800 x 259 34 and 72).  The first workgroup clears `clear`, too.
template <bool VEC>
__global__ __launch_bounds__(256) void gq_gather_w(const __half* __restrict__ W, int64_t out, int64_t in, int nr,
                                                   const int32_t* __restrict__ perm, const uint8_t* __restrict__ dead,
                                                   float* __restrict__ Wp, int32_t* __restrict__ clear, int n_clear) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_clear; i += 256) clear[i] = 0;
    extern __shared__ __align__(16) char gw_smem[];
    __half* row = reinterpret_cast<__half*>(gw_smem);
    const int64_t r0 = int64_t(blockIdx.x) * nr;
    const int n = static_cast<int>(in), rows_here = static_cast<int>(min(int64_t(nr), out - r0));
    const __half* src = W + r0 * in;
    if constexpr (VEC) {
        for (int rr = 0; rr < rows_here; ++rr)
            for (int j = threadIdx.x * 8; j < n; j += 256 * 8) {
                uint4 v = *reinterpret_cast<const uint4*>(src + rr * in + j);
                const uint2 dd = *reinterpret_cast<const uint2*>(dead + j);
                if (dd.x | dd.y) {
                    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if ((e < 4 ? dd.x >> (8 * e) : dd.y >> (8 * (e - 4))) & 0xffu) w[e / 2] &= e & 1 ? 0xffffu : 0xffff0000u;
                }
                *reinterpret_cast<uint4*>(row + rr * n + j) = v;
            }
        __syncthreads();
        for (int i = threadIdx.x * 4; i < n; i += 256 * 4) {
            const int4 p = *reinterpret_cast<const int4*>(perm + i);
            for (int rr = 0; rr < rows_here; ++rr) {
                const __half* rw = row + rr * n;
                *reinterpret_cast<float4*>(Wp + (r0 + rr) * in + i) =
                    make_float4(__half2float(rw[p.x]), __half2float(rw[p.y]), __half2float(rw[p.z]), __half2float(rw[p.w]));
            }
        }
    } else {
        // the rows follow each other in W and in LDS
        for (int j = threadIdx.x; j < rows_here * n; j += 256) row[j] = src[j];
        __syncthreads();
        if (nr == 1) {
            for (int i = threadIdx.x; i < n; i += 256) {
                const int32_t j = perm[i];
                Wp[r0 * in + i] = dead[j] ? 0.0f : __half2float(row[j]);
            }
        } else {
            for (int i = threadIdx.x; i < n; i += 256) {
                const int32_t j = perm[i];
                const bool d = dead[j] != 0;
                for (int rr = 0; rr < rows_here; ++rr) Wp[(r0 + rr) * in + i] = d ? 0.0f : __half2float(row[rr * n + j]);
            }
        }
    }
}

// visited[perm[i]] = i: where in the visiting order an original channel sits
__global__ void gq_invperm(const int32_t* __restrict__ perm, int64_t in, int32_t* __restrict__ visited) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < in) visited[perm[i]] = static_cast<int32_t>(i);
}

// codes back to the original channel order, and dW = W - scale*(code - zero) there.  nr rows per workgroup (in one row
// group per-IC: nr divides 64): their codes in visiting order are read once into LDS and looked up there; the writes
// (and the reads of W and the parameters) are consecutive.  Dynamic LDS: nr * in bytes.
// VEC: in % 8 == 0 and 16-byte aligned W, dW and parameters, 8-byte aligned codes and dead: 8 channels at a time.
// 11008 x 4096 with dW, 360 MB: 79 us, where an element at a time takes 218.  An element at a time nr is 1
// unless the rows are short and many: what counts is how many workgroups there are to hide the trips (11008 x 4090 218 us,
// with four rows per workgroup 258; 4096 x 1022 16 and 22; 38400 x 514 96 and 87; 76800 x 259 110 and 88).
template <bool IC, bool VEC>
__global__ __launch_bounds__(256) void gq_scatter(const uint8_t* __restrict__ Qp, const int32_t* __restrict__ visited,
                                                  const uint8_t* __restrict__ dead, const __half* __restrict__ W, int64_t out,
                                                  int64_t in, int nr, int g, const float* __restrict__ scales,
                                                  const uint8_t* __restrict__ zeros, int mfmt, uint8_t* __restrict__ codes,
                                                  float* __restrict__ dW) {
    extern __shared__ __align__(16) char gs_smem[];
    uint8_t* qrow = reinterpret_cast<uint8_t*>(gs_smem);
    const int64_t r0 = int64_t(blockIdx.x) * nr;
    const int n = static_cast<int>(in), rows_here = static_cast<int>(min(int64_t(nr), out - r0));
    auto param = [&](int64_t pi, float& sc, float& zp) {
        if (mfmt) {
            const uint32_t wd = reinterpret_cast<const uint16_t*>(scales)[pi];
            sc = word_scale(wd, mfmt);
            zp = word_zero(wd, mfmt);
        } else {
            sc = scales[pi];
            zp = static_cast<float>(zeros[pi]);
        }
    };
    if constexpr (VEC) {
        for (int i = threadIdx.x * 8; i < rows_here * n; i += 256 * 8)
            *reinterpret_cast<uint2*>(qrow + i) = *reinterpret_cast<const uint2*>(Qp + r0 * in + i);
        __syncthreads();
        for (int j = threadIdx.x * 8; j < n; j += 256 * 8) {
            const int4 va = *reinterpret_cast<const int4*>(visited + j), vb = *reinterpret_cast<const int4*>(visited + j + 4);
            const int vis[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
            const uint2 dd = *reinterpret_cast<const uint2*>(dead + j);
            float sc[8], zp[8];
            if (IC && dW) {
                const int64_t pi = (r0 / g) * in + j;
                if (mfmt) {
                    const uint4 m = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(scales) + pi);
                    const uint32_t mw[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t wd = (mw[e / 2] >> (16 * (e & 1))) & 0xffffu;
                        sc[e] = word_scale(wd, mfmt);
                        zp[e] = word_zero(wd, mfmt);
                    }
                } else {
                    const float4 sa = *reinterpret_cast<const float4*>(scales + pi), sb = *reinterpret_cast<const float4*>(scales + pi + 4);
                    const uint2 z = *reinterpret_cast<const uint2*>(zeros + pi);
                    sc[0] = sa.x; sc[1] = sa.y; sc[2] = sa.z; sc[3] = sa.w; sc[4] = sb.x; sc[5] = sb.y; sc[6] = sb.z; sc[7] = sb.w;
#pragma unroll
                    for (int e = 0; e < 8; ++e) zp[e] = static_cast<float>(((e < 4 ? z.x >> (8 * e) : z.y >> (8 * (e - 4))) & 0xffu));
                }
            }
            for (int rr = 0; rr < rows_here; ++rr) {
                const int64_t idx = (r0 + rr) * in + j;
                uint32_t q[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] = qrow[rr * n + vis[e]];
                *reinterpret_cast<uint2*>(codes + idx) = make_uint2(q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24),
                                                                    q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24));
                if (!dW) continue;
                if constexpr (!IC) {
                    const int64_t p0 = (r0 + rr) * (n / g);
                    if ((g & 7) == 0) {                       // one group for the eight
                        param(p0 + j / g, sc[0], zp[0]);
#pragma unroll
                        for (int e = 1; e < 8; ++e) { sc[e] = sc[0]; zp[e] = zp[0]; }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) param(p0 + (j + e) / g, sc[e], zp[e]);
                    }
                }
                const uint4 raw = *reinterpret_cast<const uint4*>(W + idx);
                const __half2* h = reinterpret_cast<const __half2*>(&raw);
                float d[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float w = (e < 4 ? dd.x >> (8 * e) : dd.y >> (8 * (e - 4))) & 0xffu ? 0.0f
                                    : e & 1 ? __high2float(h[e / 2]) : __low2float(h[e / 2]);
                    const float wq = sc[e] * (static_cast<float>(q[e]) - zp[e]);
                    d[e] = w - wq;
                }
                float4* dst = reinterpret_cast<float4*>(dW + idx);
                dst[0] = make_float4(d[0], d[1], d[2], d[3]);
                dst[1] = make_float4(d[4], d[5], d[6], d[7]);
            }
        }
    } else {
        for (int i = threadIdx.x; i < rows_here * n; i += 256) qrow[i] = Qp[r0 * in + i];
        __syncthreads();
        for (int rr = 0; rr < rows_here; ++rr)
            for (int j = threadIdx.x; j < n; j += 256) {
                const int64_t r = r0 + rr, idx = r * in + j;
                const uint8_t q = qrow[rr * n + visited[j]];
                codes[idx] = q;
                if (dW) {
                    float sc, zp;
                    param(IC ? (r / g) * in + j : r * (in / g) + j / g, sc, zp);
                    const float wq = sc * (static_cast<float>(q) - zp);
                    dW[idx] = (dead[j] ? 0.0f : __half2float(W[idx])) - wq;
                }
            }
    }
}

// The next block's columns [col0, col0 + w), w <= 128: the same update, for the launch that two sweeps wait for.  A
// thread takes RT rows of one column and has the column's next sixteen entries of U on their way while it works on
// sixteen: the launch is short of waves, so what counts is that few trips to memory follow each other.
template <int RT>
__global__ __launch_bounds__(256) void gq_next(float* __restrict__ Wp, const float* __restrict__ U, const float* __restrict__ Ep,
                                               int64_t out, int64_t in, int64_t i1, int64_t col0, int w) {
    constexpr int KB = 16;
    __shared__ __align__(16) float Es[GB][2 * RT];            // [channel][row]
    __builtin_amdgcn_s_setprio(2);                            // a link of the chain, as the sweep
    const int c = threadIdx.x & (GB - 1), rq = (threadIdx.x >> 7) * RT;
    const int64_t r0 = int64_t(blockIdx.x) * (2 * RT), jj = col0 + min(c, w - 1);
    float u[2][KB], t[RT], v[RT];
    const float* urow = U + i1 * in;                          // the row to fetch next
    auto fetch = [&](int b) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            u[b][kk] = urow[static_cast<uint32_t>(jj)];
            urow += in;
        }
        asm volatile("" ::: "memory");                        // issued here, and the reads of Es below not above
    };
    auto step = [&](int b, int k) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
#pragma unroll
            for (int i = 0; i < RT; i += 4) {
                const float4 e = *reinterpret_cast<const float4*>(&Es[k + kk][rq + i]);
                const float e4[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float upd = e4[r] * u[b][kk];
                    v[i + r] = v[i + r] - upd;
                }
            }
            if (kk % 4 == 3) asm volatile("" ::: "memory");   // (or all of Es's entries would be read first)
        }
    };
    fetch(0);
#pragma unroll
    for (int q = 0; q < RT; ++q) t[q] = Ep[min(r0 + rq + q, out - 1) * in + i1 + c];
#pragma unroll
    for (int r = 0; r < RT; ++r) v[r] = Wp[min(r0 + rq + r, out - 1) * in + jj];
#pragma unroll
    for (int q = 0; q < RT; ++q) Es[c][rq + q] = t[q];
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < GB; k += 2 * KB) {
        fetch(1);
        step(0, k);
        if (k + 2 * KB < GB) fetch(0);
        step(1, k + KB);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r)
        if (c < w && r0 + rq + r < out) Wp[(r0 + rq + r) * in + jj] = v[r];
}

}  // namespace

int launch_gptq_prepare(adadim_ctx* ctx, const float* H, int64_t n, float percdamp, int act_order, int32_t* perm,
                        uint8_t* dead, float* U) {
    const size_t mat = size_t(n) * size_t(n) * sizeof(double);
    double* A = static_cast<double*>(adadim_workspace(ctx, WS_GPTQ_A, mat));
    double* M = static_cast<double*>(adadim_workspace(ctx, WS_GPTQ_M, mat));
    double* dvec = static_cast<double*>(adadim_workspace(ctx, WS_GPTQ_D, size_t(n + 1) * sizeof(double)));
    double* T = static_cast<double*>(adadim_workspace(ctx, WS_GPTQ_T, FACTOR_T_ELEMS * sizeof(double)));
    int32_t* rank = static_cast<int32_t*>(adadim_workspace(ctx, WS_GPTQ_V, size_t(n) * sizeof(int32_t)));   // free here
    if (!A || !M || !dvec || !T || !rank) return ADADIM_EHIP;
    double* damp = dvec + n;
    const unsigned nb1 = static_cast<unsigned>((n + 255) / 256), nb2 = static_cast<unsigned>((n * n + 255) / 256);
    ProfScope prof(ctx, "gptq_prepare");
    hipLaunchKernelGGL(gq_diag, dim3(nb1), dim3(256), 0, ctx->stream, H, n, dvec, dead);
    hipLaunchKernelGGL(gq_damp, dim3(1), dim3(256), 0, ctx->stream, dvec, n, static_cast<double>(percdamp), damp);
    if (act_order) {
        hipLaunchKernelGGL(gq_zero_i32, dim3(nb1), dim3(256), 0, ctx->stream, rank, n);
        hipLaunchKernelGGL(gq_rank_count, dim3(nb1, static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, ctx->stream,
                           dvec, n, rank);
        hipLaunchKernelGGL(gq_rank_place, dim3(nb1), dim3(256), 0, ctx->stream, rank, n, perm);
    } else
        hipLaunchKernelGGL(gq_rank, dim3(nb1), dim3(256), 0, ctx->stream, dvec, n, act_order, perm);
    if (n <= 16384)                                           // 64 KB of LDS
        hipLaunchKernelGGL(gq_gather, dim3(static_cast<unsigned>(n)), dim3(256), static_cast<size_t>(n) * 4, ctx->stream, H, n, perm,
                           dvec, damp, A);
    else
        hipLaunchKernelGGL(gq_gather_wide, dim3(nb2), dim3(256), 0, ctx->stream, H, n, perm, dvec, damp, A);
    ADADIM_LAUNCH_CHECK(ctx, "gptq prepare");
    static_assert(GT == NB, "the first tile of a step or an update is the next diagonal block");
    FactorPlan(n).run([&](const FactorLaunch& l) {
        // the jobs in further rows of workgroups (at most 52000, for 46340 channels and one column)
        const unsigned cols = static_cast<unsigned>(l.cols), tiles = static_cast<unsigned>(l.jobs.tiles());
        const dim3 grid(cols, static_cast<unsigned>(l.rows) + (cols > 0 ? (tiles + cols - 1) / cols : 0));
        switch (l.kind) {
            case FACTOR_DIAG:
                hipLaunchKernelGGL(chol_diag_inv, dim3(1), dim3(256), 0, ctx->stream, A, M, n, l.k0, l.w);
                break;
            case FACTOR_STEP:
                hipLaunchKernelGGL(chol_step, grid, dim3(256), 0, ctx->stream, A, M, T, U, n, l.k0, l.rows, l.jobs);
                break;
            case FACTOR_BELOW:
                hipLaunchKernelGGL(chol_panel, dim3(static_cast<unsigned>(l.rows)), dim3(256), 0, ctx->stream, A, M, n, l.k0, l.w);
                break;
            case FACTOR_UPDATE:
                hipLaunchKernelGGL(chol_syrk_diag, grid, dim3(256), 0, ctx->stream, A, M, T, U, n, l.k0, l.w, l.k1, l.rows, l.jobs);
                break;
            default:
                hipLaunchKernelGGL(factor_jobs, dim3(tiles), dim3(256), 0, ctx->stream, A, M, T, U, n, l.jobs);
        }
    });
    ADADIM_LAUNCH_CHECK(ctx, "gptq factor");
    return ADADIM_OK;
}

int launch_gptq_quantize(adadim_ctx* ctx, const __half* W, int64_t out, int64_t in, int dim, int bits, int g,
                         const float* U, const int32_t* perm, const uint8_t* dead, const float* st_scales,
                         const uint8_t* st_zeros, uint8_t* codes, float* scales_out, uint8_t* zeros_out, float* dW,
                         int mfmt) {
    const size_t mat = size_t(out) * size_t(in) * sizeof(float);
    float* Wp = static_cast<float*>(adadim_workspace(ctx, WS_GPTQ_W, mat));
    const bool ic = dim == ADADIM_DIM_IC;
    const bool whole = !ic && rows::better(out, in);          // per-OC, the whole sweep in one launch
    // (not used by a whole sweep; with it, whether a sweep can be recorded after another depends on their sizes alone)
    float* Ep = static_cast<float*>(adadim_workspace(ctx, WS_GPTQ_E, mat));
    uint8_t* Qp = static_cast<uint8_t*>(adadim_workspace(ctx, WS_GPTQ_Q, size_t(out) * size_t(in)));
    int32_t* visited = static_cast<int32_t*>(adadim_workspace(ctx, WS_GPTQ_V, size_t(in) * sizeof(int32_t)));
    if (!Wp || !Ep || !Qp || !visited) return ADADIM_EHIP;
    const float qmax = static_cast<float>((1 << bits) - 1);
    static PerDeviceOnce once;
    ADADIM_HIP_TRY(ctx, once.run([] {
        hipError_t e = groups::allow_lds();
        if (e == hipSuccess) e = rows::allow_lds();
        if (e == hipSuccess) e = blocks::allow_lds();
        // rows of W in LDS: 64 KB of them, or one of up to 46340 halves
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(gq_gather_w<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    96 * 1024);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(gq_gather_w<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    96 * 1024);
        return e;
    }));
    // per-IC: a counter per block's launch, in the room of `visited`, which is filled in behind the sweep
    const int n_blocks = ic ? static_cast<int>((in + GB - 1) / GB) : 0;
    {
        ProfScope prof(ctx, "gptq_gather");
        // up to four rows per workgroup, as long as four workgroups fit a compute unit's LDS and the chip stays full
        const bool vec = (in & 7) == 0 && aligned16(W) && aligned16(perm) && (reinterpret_cast<uintptr_t>(dead) & 7u) == 0;
        const int nr = in <= 5000 && out >= 4096 ? 4 : in <= 10000 && out >= 2048 ? 2 : 1;
        const dim3 grid(static_cast<unsigned>((out + nr - 1) / nr));
        const size_t lds_bytes = size_t(nr) * size_t(in) * 2;
        if (vec) hipLaunchKernelGGL(gq_gather_w<true>, grid, dim3(256), lds_bytes, ctx->stream, W, out, in, nr, perm, dead, Wp, visited, n_blocks);
        else hipLaunchKernelGGL(gq_gather_w<false>, grid, dim3(256), lds_bytes, ctx->stream, W, out, in, nr, perm, dead, Wp, visited, n_blocks);
    }
    if (whole) {
        ProfScope prof(ctx, "gptq_sweep");
        const int r = rows::rows_per_group(out, in);
        const dim3 grid(static_cast<unsigned>((out + r - 1) / r));
#define GQ_ROWS(R)                                                                                                      \
    case R:                                                                                                             \
        hipLaunchKernelGGL(rows::gq_rows<R>, grid, dim3(64 * rows::WAVES), sizeof(rows::Lds<R>), ctx->stream, Wp, U, perm, \
                           out, in, g, qmax, mfmt, st_scales, st_zeros, Qp);                                            \
        break
        switch (r) {
            GQ_ROWS(4);
            GQ_ROWS(8);
            GQ_ROWS(12);
            GQ_ROWS(16);
            GQ_ROWS(24);
            GQ_ROWS(32);
        }
#undef GQ_ROWS
    }
    for (int64_t i1 = 0; ic && i1 < in; i1 += GB) {
        ProfScope prof(ctx, "gptq_sweep");
        const int nbw = static_cast<int>(in - i1 < GB ? in - i1 : GB);
        const int64_t n_groups = out / g, n_items = n_groups + groups::n_pieces(out, in, i1);
        const dim3 grid(static_cast<unsigned>(std::min<int64_t>(n_items, 256)));
#define GQ_GO(RPL)                                                                                                       \
    hipLaunchKernelGGL(groups::gq_group_step<RPL>, grid, dim3(64 * groups::WAVES), sizeof(groups::Lds<RPL>), ctx->stream, Wp, U, perm, in, \
                       i1, nbw, static_cast<int>(n_groups), static_cast<int>(n_items), qmax, 1.0f / qmax, mfmt, scales_out, \
                       zeros_out, Qp, Ep, visited + i1 / GB)
        if (g == 64) GQ_GO(1);
        else GQ_GO(2);
#undef GQ_GO
    }
    // Per-OC a launch per block for the walk alone: a block's errors reach the channels behind it in two launches: the next block's
    // 128 channels at once, on the main stream, so that the next sweep can start; the rest on a side stream, under
    // that sweep.  Every element still receives the
    // blocks' errors in block order: the side stream applies them in order, and the main stream
    // waits for the side stream's last launch before it adds the following block's errors to the
    // channels that launch wrote.  With per-kernel timing on, everything runs on the main stream.
    const bool by_block = !ic && !whole;
    const bool overlap = by_block && !ctx->prof.enabled && in > 2 * GB;
    if (overlap && !adadim_side_stream(ctx)) return ADADIM_EHIP;
    bool side_busy = false;
    for (int64_t i1 = 0; by_block && i1 < in; i1 += GB) {
        const int nbw = static_cast<int>(in - i1 < GB ? in - i1 : GB);
        {
            ProfScope prof(ctx, "gptq_sweep");
            hipLaunchKernelGGL(blocks::gq_block, dim3(static_cast<unsigned>((out + blocks::ROWS - 1) / blocks::ROWS)), dim3(256),
                               sizeof(blocks::Lds), ctx->stream, Wp, U, perm, out, in, i1, nbw, g, qmax, mfmt, st_scales, st_zeros, Qp, Ep);
        }
        const int64_t behind = i1 + nbw;                        // first channel behind the block
        if (behind >= in) break;
        const int64_t next_end = behind + GB < in ? behind + GB : in;
        auto trailing = [&](hipStream_t stream, int64_t col0) {
            const bool narrow = in - col0 <= update::COLS_NARROW;
            const dim3 grid(narrow ? 1 : static_cast<unsigned>((in - col0 + update::COLS - 1) / update::COLS),
                            static_cast<unsigned>((out + update::ROWS - 1) / update::ROWS));
            hipLaunchKernelGGL(narrow ? update::gq_trailing<true> : update::gq_trailing<false>, grid, dim3(256), 0, stream, Wp, U, Ep, out, in,
                               i1, col0, in);
        };
        if (!overlap) {
            ProfScope prof(ctx, "gptq_trailing");
            trailing(ctx->stream, behind);
            continue;
        }
        if (side_busy) ADADIM_HIP_TRY(ctx, hipStreamWaitEvent(ctx->stream, ctx->side_ev[1], 0));
        hipLaunchKernelGGL(gq_next<4>, dim3(static_cast<unsigned>((out + 7) / 8)), dim3(256), 0, ctx->stream, Wp, U, Ep, out, in, i1,
                           behind, static_cast<int>(next_end - behind));
        // the side stream starts behind this short launch, not beside it: the next sweep waits for it
        ADADIM_HIP_TRY(ctx, hipEventRecord(ctx->side_ev[0], ctx->stream));
        if (next_end < in) {
            ADADIM_HIP_TRY(ctx, hipStreamWaitEvent(ctx->side, ctx->side_ev[0], 0));
            trailing(ctx->side, next_end);
            ADADIM_HIP_TRY(ctx, hipEventRecord(ctx->side_ev[1], ctx->side));
            side_busy = true;
        }
    }
    if (side_busy) ADADIM_HIP_TRY(ctx, hipStreamWaitEvent(ctx->stream, ctx->side_ev[1], 0));   // join
    {
        ProfScope prof(ctx, "gptq_scatter");
        hipLaunchKernelGGL(gq_invperm, dim3(static_cast<unsigned>((in + 255) / 256)), dim3(256), 0, ctx->stream, perm, in,
                           visited);
        const float* sc = ic ? scales_out : st_scales;
        const uint8_t* zp = ic ? zeros_out : st_zeros;
        const bool vec = (in & 7) == 0 && aligned16(W) && aligned16(dW) && (reinterpret_cast<uintptr_t>(dead) & 7u) == 0 &&
                         (reinterpret_cast<uintptr_t>(codes) & 7u) == 0 &&
                         (!ic || (aligned16(sc) && (reinterpret_cast<uintptr_t>(zp) & 7u) == 0));
        const bool share = vec ? in <= 10000 && out >= 4096 : in <= 128 ? out >= 4096 : in <= 600 && out >= 8192;
        const int nr = share ? 4 : 1;                                          // (divides a per-IC group)
        const dim3 grid(static_cast<unsigned>((out + nr - 1) / nr));
        const size_t lds_bytes = size_t(nr) * size_t(in);
#define GQ_SC(IC, VEC)                                                                                                   \
    hipLaunchKernelGGL((gq_scatter<IC, VEC>), grid, dim3(256), lds_bytes, ctx->stream, Qp, visited, dead, W, out, in, nr, g, sc, \
                       zp, mfmt, codes, dW)
        if (ic) { if (vec) GQ_SC(true, true); else GQ_SC(true, false); }
        else { if (vec) GQ_SC(false, true); else GQ_SC(false, false); }
#undef GQ_SC
    }
    ADADIM_LAUNCH_CHECK(ctx, "gptq sweep");
    return ADADIM_OK;
}
