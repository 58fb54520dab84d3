// De-quantizing matrix-vector product for per-IC quantized weights (paper Sec. 4.5, App. D):
//     y[o] = sum_j scale[o/g, j] * (code[o, j] - zero[o/g, j]) * x[j]
// from the packed stream adadim_quantize(dim = IC) writes: [in, out*b/32] words, the codes of
// one input column consecutive along the output axis.  Batch 1: every weight bit is read once
// and used once, so the kernel is bound by HBM reads.
//
// The paper's kernel builds look-up tables of scale*activation products; on gfx950 a direct
// form is simpler and reads the same bytes: with a[r, j] = scale[r, j] * x[j] (the per-IC
// scale folded into the activation, as the paper does when it fills its tables)
//     y[o] = sum_j a[o/g, j] * code[o, j]  -  sum_j a[o/g, j] * zero[o/g, j].
// A lane owns 32 consecutive outputs (b words of every column, one 16-byte load for b = 4); LO lanes of a wavefront lie
// along the outputs, so that a column is read in pieces of LO * 4b bytes, and its other 64 / LO lanes take other
// columns.  The second sum costs one fma per lane and column.  Columns are split over the lanes, the eight waves of a
// block and over blocks; partial outputs are added up in a fixed order (LDS inside a block; across blocks by the block
// of an output tile that finishes last, part by part), so the result is reproducible.  The split is gemv_plan.h's.
//
// How the last block sees the others' partial sums: they are stored and loaded as relaxed atomics at device scope, which
// on this chip go past the XCD's L2 (to the memory side, where all XCDs meet), a block waits for its stores before it
// takes its ticket, and only partial sums travel this way.  (Plain stores with device-scope fences write back and
// invalidate the XCD's whole L2, where x and the group parameters live: 3x slower overall.  A second launch for the
// sum cost 4-6 us of a call, as much as the product of a 4096 x 4096 layer.)
#include "common.h"
#include "code_fields.h"
#include "gemv_plan.h"

namespace {

constexpr int GV_NBUF = 3;                 // load buffers taken in turn (4 to 6 were measured: no faster)

template <int PB>
struct Words {
    uint32_t w[PB];
};

// STREAM: past the caches as far as can be said.  With ranges a compute unit's waves hold 16 groups' parameters each, as much
// as its first-level cache takes, and the code words that pass through push them out between two steps: 49152 x 12288,
// 4 bits, 66.6 us without, 63.9 with; 151552 x 4096, 3 bits, 58.0 and 56.1.  With turns it loses (14336 x 4096 12.7 and 13.2).
template <int PB, bool STREAM>
__device__ __forceinline__ Words<PB> load_words(const uint32_t* p) {
    typedef uint32_t Vec __attribute__((ext_vector_type(PB == 3 ? 1 : PB)));
    constexpr int N = PB == 3 ? 1 : PB;                       // words per load
    Words<PB> r;
#pragma unroll
    for (int i = 0; i < PB; i += N) {
        const Vec* at = reinterpret_cast<const Vec*>(p + i);
        Vec v;
        if constexpr (STREAM) v = __builtin_nontemporal_load(at);
        else v = *at;
#pragma unroll
        for (int e = 0; e < N; ++e) r.w[i + e] = v[e];
    }
    return r;
}

// float(byte n of v)
__device__ __forceinline__ float ubyte(uint32_t v, int n) { return static_cast<float>((v >> (8 * n)) & 0xffu); }
// the value in a vector register, opaque to the optimiser (a constant stays a register operand)
__device__ __forceinline__ uint32_t hide(uint32_t v) {
    asm("" : "+v"(v));
    return v;
}
// (v & mask) | orc in one instruction: the encoding takes one scalar operand, so the mask travels in a scalar
// register and the or-constant in a vector register (see hide()); left alone the compiler emits an and and an or,
// each with a literal
__device__ __forceinline__ uint32_t and_or(uint32_t v, uint32_t mask, uint32_t orc) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(mask), "v"(orc));
    return r;
}

__device__ __forceinline__ __half2 as_half2(uint32_t v) { return *reinterpret_cast<const __half2*>(&v); }
// acc[k] += a * (code k of the lane's 32 codes + code_offset(k)): the plan of code_fields.h, unrolled.  The
// exponent constants sit in vector registers, the masks become scalar operands (see and_or).
template <int PB>
__device__ __forceinline__ void accumulate(const Words<PB>& wd, float a, float (&acc)[32]) {
    static_assert(PB >= 2 && PB <= 4, "2, 3 or 4 bits");
    constexpr int NS = field_steps<PB>(), NO = field_orcs<PB>();
    uint32_t orc[NO];
#pragma unroll
    for (int q = 0; q < NO; ++q) orc[q] = hide(field_orc<PB>(q));
    // the words as stored and shifted: per word for 4 and 2 bits (by 8, by 10), across words for 3 bits (by 8)
    uint32_t src[PB][2];
#pragma unroll
    for (int w = 0; w < PB; ++w) {
        src[w][0] = wd.w[w];
        if constexpr (PB == 3) src[w][1] = w + 1 < PB ? __builtin_amdgcn_alignbit(wd.w[w + 1 < PB ? w + 1 : w], wd.w[w], 8) : wd.w[w] >> 8;
        else src[w][1] = wd.w[w] >> (PB == 4 ? 8 : 10);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const FieldStep f = field_step<PB>(s);
        const __half2 h = as_half2(and_or(src[f.word][f.shift != 0], f.mask, orc[f.orc_id]));
        if (f.k_lo >= 0) acc[f.k_lo] = fmaf(__low2float(h), a, acc[f.k_lo]);
        if (f.k_hi >= 0) acc[f.k_hi] = fmaf(__high2float(h), a, acc[f.k_hi]);
    }
}

// M16: the group parameters come as one 16-bit word per (group, column) in `scales` (the
// fp16 pattern of the scale without its sign bit and its PB-1 lowest bits, above the PB-bit
// zero-point) instead of an fp32 scale and a u8 zero-point.
template <int PB, bool M16, int LO, bool RANGES>
__global__ __launch_bounds__(64 * GV_WAVES, 4) void gemv_ic_tiles(const uint32_t* __restrict__ packed,
                                                               const void* __restrict__ scales,
                                                               const uint8_t* __restrict__ zeros,
                                                               const __half* __restrict__ x, int64_t out, int64_t in,
                                                               int g, int64_t n_words, float* part,
                                                               unsigned int* ticket, __half* __restrict__ y) {
    constexpr int CL = 64 / LO;                               // column lanes
    constexpr int NP = RANGES ? CL : 1;                     // partial sums of an output that the block leaves
    __shared__ float s_acc[GV_WAVES][32][65];
    __shared__ unsigned int s_ticket;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cl = lane / LO;
    const int64_t tile0 = int64_t(blockIdx.x) * (LO * 32);
    const int64_t o_lane = tile0 + (lane % LO) * 32;
    const bool valid = o_lane < out;                         // out % 32 == 0: a lane's outputs are inside together
    // (32-bit divisions: out and in are below 2^24)
    const int64_t r = valid ? static_cast<uint32_t>(o_lane) / static_cast<uint32_t>(g) : 0;
    const GemvColumns<LO, RANGES> cols(in, gridDim.y, blockIdx.y, wave, cl);
    const uint32_t* wp = packed + (valid ? (o_lane >> 5) * PB : 0);
    float acc[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) acc[k] = 0.0f;
    float zsum = 0.0f, asum = 0.0f;                           // sums of a * zero and of a
    // four columns per step, the next step's loads issued before this step's arithmetic
    struct Step {
        Words<PB> wd[4];
        float4 s4;
        uint32_t z4;
        uint2 m4;
        uint2 xr;
        bool have;
    };
    auto fetch = [&](Step& st, int step) {
        const int64_t j0 = int64_t(cols.quad(step)) * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) st.wd[c] = load_words<PB, RANGES>(wp + (j0 + c) * n_words);
        if constexpr (M16) {
            st.m4 = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(scales) + r * in + j0);
        } else {
            st.s4 = *reinterpret_cast<const float4*>(static_cast<const float*>(scales) + r * in + j0);
            st.z4 = *reinterpret_cast<const uint32_t*>(zeros + r * in + j0);
        }
        st.xr = *reinterpret_cast<const uint2*>(x + j0);
        st.have = cols.has(step);
    };
    auto consume = [&](const Step& st) {
        const float2 x01 = __half22float2(*reinterpret_cast<const __half2*>(&st.xr.x));
        const float2 x23 = __half22float2(*reinterpret_cast<const __half2*>(&st.xr.y));
        float a[4], z[4];
        if constexpr (M16) {
            // both words of a register at once: shifted right by one, the kept pattern bits of each
            // word land on their fp16 positions and the mask clears what crossed over
            constexpr uint32_t KEEP = (0x7FFFu & ~((1u << (PB - 1)) - 1u)) * 0x10001u, ZM = (1u << PB) - 1u;
            const uint32_t h01 = (st.m4.x >> 1) & KEEP, h23 = (st.m4.y >> 1) & KEEP;
            const float2 s01 = __half22float2(*reinterpret_cast<const __half2*>(&h01));
            const float2 s23 = __half22float2(*reinterpret_cast<const __half2*>(&h23));
            a[0] = s01.x * x01.x; a[1] = s01.y * x01.y; a[2] = s23.x * x23.x; a[3] = s23.y * x23.y;
            z[0] = static_cast<float>(st.m4.x & ZM); z[1] = static_cast<float>((st.m4.x >> 16) & ZM);
            z[2] = static_cast<float>(st.m4.y & ZM); z[3] = static_cast<float>((st.m4.y >> 16) & ZM);
        } else {
            a[0] = st.s4.x * x01.x; a[1] = st.s4.y * x01.y; a[2] = st.s4.z * x23.x; a[3] = st.s4.w * x23.y;
#pragma unroll
            for (int c = 0; c < 4; ++c) z[c] = ubyte(st.z4, c);
        }
        if constexpr (CL > 1) {
#pragma unroll
            for (int c = 0; c < 4; ++c) a[c] = st.have ? a[c] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            zsum = fmaf(a[c], z[c], zsum);
            asum += a[c];
            accumulate<PB>(st.wd[c], a[c], acc);
        }
    };
    const int trips = static_cast<int>(cols.trips);
    if (valid && trips > 0) {
        // GV_NBUF buffers taken in turn, no copies: one is consumed while the others are in flight (a step is 2 to
        // 4 KB per wave; the memory system wants several of them outstanding per wave).  Fetches past the end
        // re-read the share's last step and are not consumed.
        Step st[GV_NBUF];
#pragma unroll
        for (int b = 0; b < GV_NBUF - 1; ++b) fetch(st[b], min(b, trips - 1));
        for (int s0 = 0; s0 < trips; s0 += GV_NBUF) {
#pragma unroll
            for (int b = 0; b < GV_NBUF; ++b) {
                fetch(st[(b + GV_NBUF - 1) % GV_NBUF], min(s0 + b + GV_NBUF - 1, trips - 1));
                if (s0 + b < trips) consume(st[b]);
            }
        }
    }
    // OFFSET: the codes were read as code + code_offset(k)
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        s_acc[wave][k][lane] = (acc[k] - code_offset<PB>(k) * asum) - zsum;
    }
    __syncthreads();
    // thread t adds up the waves (and, without ranges, the column lanes) for outputs t, t + 512, .. of the block's LO * 32
    // (consecutive threads consecutive outputs: what goes past the caches goes in whole lines)
    constexpr int STEP = 64 * GV_WAVES, OPT = LO * 32 > STEP ? LO * 32 / STEP : 1;
    const int t = threadIdx.x;
    const int n_out = static_cast<int>(min(int64_t(LO * 32), out - tile0));
    float v[OPT], sums[NP][OPT];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int e = 0; e < OPT; ++e) {
            const int ol = t + STEP * e, ln = (ol >> 5) % LO, k = ol & 31;
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < GV_WAVES; ++w)
#pragma unroll
                for (int c = 0; c < CL / NP; ++c) sum += s_acc[w][k][(p + c) * LO + ln];
            sums[p][e] = sum;
        }
    if (gridDim.y > 1) {
        float* const mine = part + int64_t(blockIdx.y) * NP * out + tile0;
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int e = 0; e < OPT; ++e)
                if (t + STEP * e < n_out)
                    __hip_atomic_store(mine + p * out + t + STEP * e, sums[p][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // every wave's partial sums have arrived ...
        __syncthreads();
        if (t == 0) s_ticket = __hip_atomic_fetch_add(ticket + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_ticket != gridDim.y - 1) return;                // ... before the block counts itself in
        if (t == 0) __hip_atomic_store(ticket + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t >= n_out) return;
#pragma unroll
        for (int e = 0; e < OPT; ++e) v[e] = 0.0f;
        const float* const src = part + tile0;
        const unsigned n_parts = gridDim.y * NP;
        for (unsigned c0 = 0; c0 < n_parts; c0 += 8) {        // eight parts' loads in flight
            float p[8][OPT];
#pragma unroll
            for (unsigned c = 0; c < 8; ++c)
#pragma unroll
                for (int e = 0; e < OPT; ++e)
                    p[c][e] = c0 + c < n_parts && (e == 0 || t + STEP * e < n_out)
                                  ? __hip_atomic_load(src + int64_t(c0 + c) * out + t + STEP * e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                  : 0.0f;
#pragma unroll
            for (unsigned c = 0; c < 8; ++c)
#pragma unroll
                for (int e = 0; e < OPT; ++e) v[e] += p[c][e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < OPT; ++e) {
            v[e] = 0.0f;
#pragma unroll
            for (int p = 0; p < NP; ++p) v[e] += sums[p][e];
        }
    }
#pragma unroll
    for (int e = 0; e < OPT; ++e)
        if (t + STEP * e < n_out) y[tile0 + t + STEP * e] = __float2half_rn(v[e]);
}

// Counters of the output tiles (one each; a tile of several blocks is one of at most GV_SLOTS), zero between launches: the
// block that finds itself last clears its own.
constexpr size_t GV_COUNTERS = GV_SLOTS * sizeof(unsigned int);
__global__ void gemv_zero(unsigned int* counters) { counters[threadIdx.x] = 0u; }

// WS_GEMV_PART with room for the counters and `bytes` behind them, or nullptr.
char* gemv_slot(adadim_ctx* ctx, size_t bytes) { return static_cast<char*>(adadim_workspace(ctx, WS_GEMV_PART, GV_COUNTERS + bytes)); }

// Measurement aid: the same code words read by the same grid, waves and column ranges as gemv_ic_tiles, with one
// xor per word in place of the arithmetic and no parameters, x, LDS reduction or partial sums: what the kernel's
// access pattern alone costs.  Each thread leaves one word in `sink` so that the loads are not dropped.
template <int PB, int LO, bool RANGES>
__global__ __launch_bounds__(64 * GV_WAVES, 4) void gemv_bare_read(const uint32_t* __restrict__ packed, int64_t out,
                                                                int64_t in, int64_t n_words,
                                                                uint32_t* __restrict__ sink) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cl = lane / LO;
    const int64_t o_lane = int64_t(blockIdx.x) * (LO * 32) + (lane % LO) * 32;
    const bool valid = o_lane < out;
    const GemvColumns<LO, RANGES> cols(in, gridDim.y, blockIdx.y, wave, cl);
    const uint32_t* wp = packed + (valid ? (o_lane >> 5) * PB : 0);
    uint32_t acc = 0;
    if (valid) {
        for (uint32_t s = 0; s < cols.trips; ++s) {
            const int64_t j0 = int64_t(cols.quad(s)) * 4;
            Words<PB> wd[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) wd[c] = load_words<PB, RANGES>(wp + (j0 + c) * n_words);
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int w = 0; w < PB; ++w) acc ^= wd[c].w[w];
        }
    }
    sink[(int64_t(blockIdx.y) * gridDim.x + blockIdx.x) * (64 * GV_WAVES) + threadIdx.x] = acc;
}

}  // namespace

extern "C" int adadim_probe_gemv_read(adadim_ctx* ctx, const void* packed, int64_t out, int64_t in, int bits,
                                      double* us) {
    if (!ctx) return ADADIM_ENULL;
    if (!packed || !us) return adadim_fail(ctx, ADADIM_ENULL, "adadim_probe_gemv_read: NULL argument");
    if (bits < 2 || bits > 4 || out <= 0 || in <= 0 || out > (int64_t(1) << 24) || in > (int64_t(1) << 24) ||
        (out % 32) != 0 || (in % 4) != 0)
        return adadim_fail(ctx, ADADIM_EINVAL, "adadim_probe_gemv_read: bits 2..4, out a multiple of 32, in of 4, both "
                                               "at most 2^24");
    if (reinterpret_cast<uintptr_t>(packed) & 15u)
        return adadim_fail(ctx, ADADIM_EALIGN, "adadim_probe_gemv_read: packed must be 16-byte aligned");
    if (ctx->capturing) return adadim_fail(ctx, ADADIM_EINVAL, "adadim_probe_gemv_read: not while a graph is being recorded");
    const GemvPlan sh = gemv_plan(out, in, bits, 128, false);   // as launch_gemv_ic with fp32 scales of groups of 128
    char* slot = gemv_slot(ctx, size_t(sh.tiles) * size_t(sh.chunks) * 64 * GV_WAVES * sizeof(uint32_t));
    if (!slot) return ADADIM_EHIP;
    uint32_t* sink = reinterpret_cast<uint32_t*>(slot + GV_COUNTERS);
    const int64_t n_words = out * bits / 32;
    const dim3 grid(static_cast<unsigned>(sh.tiles), static_cast<unsigned>(sh.chunks));
    hipEvent_t e0, e1;
    ADADIM_HIP_TRY(ctx, hipEventCreate(&e0));
    ADADIM_HIP_TRY(ctx, hipEventCreate(&e1));
    ADADIM_HIP_TRY(ctx, hipEventRecord(e0, ctx->stream));
    const uint32_t* pk = static_cast<const uint32_t*>(packed);
#define GV_LO(GO, PB)                         \
    switch (sh.lo) {                           \
        case 8: GO(PB, 8, false); break;       \
        case 16: GO(PB, 16, false); break;     \
        case 32: GO(PB, 32, false); break;     \
        default: GO(PB, 64, true); break;      \
    }
#define GV_PB(GO)                                                        \
    if (sh.lo == 32 && sh.ranges) GO(4, 32, true); /* four bits alone */ \
    else switch (bits) {                                                 \
        case 2: GV_LO(GO, 2) break;                                      \
        case 3: GV_LO(GO, 3) break;                                      \
        default: GV_LO(GO, 4) break;                                     \
    }
#define GV_READ(PB, LO, RANGES) hipLaunchKernelGGL((gemv_bare_read<PB, LO, RANGES>), grid, dim3(64 * GV_WAVES), 0, ctx->stream, pk, out, in, n_words, sink)
    GV_PB(GV_READ)
#undef GV_READ
    const hipError_t le = hipGetLastError();
    hipError_t e = hipEventRecord(e1, ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (le != hipSuccess) return adadim_fail(ctx, ADADIM_EHIP, "adadim_probe_gemv_read: launch: %s", hipGetErrorString(le));
    if (e != hipSuccess) return adadim_fail(ctx, ADADIM_EHIP, "adadim_probe_gemv_read: %s", hipGetErrorString(e));
    *us = double(ms) * 1e3;
    return ADADIM_OK;
}

int launch_gemv_ic(adadim_ctx* ctx, const uint32_t* packed, const void* scales, const uint8_t* zeros, const __half* x,
                   int64_t out, int64_t in, int bits, int g, __half* y, bool meta16) {
    const GemvPlan sh = gemv_plan(out, in, bits, g, meta16);
    // Room for the partial sums of whole rounds of 64-lane tiles, which no form exceeds: whether a product can be recorded
    // after another has run depends on their sizes alone.
    char* slot = gemv_slot(ctx, size_t(gemv_round_parts(out, in)) * size_t(out) * sizeof(float));
    if (!slot) return ADADIM_EHIP;
    unsigned int* ticket = reinterpret_cast<unsigned int*>(slot);
    float* part = reinterpret_cast<float*>(slot + GV_COUNTERS);
    if (sh.chunks > 1 && ctx->gemv_ready_bytes != ctx->ws_bytes[WS_GEMV_PART]) {
        hipLaunchKernelGGL(gemv_zero, dim3(1), dim3(GV_SLOTS), 0, ctx->stream, ticket);
        ADADIM_LAUNCH_CHECK(ctx, "gemv_zero");
        // a clearing that is only recorded has not happened yet for the calls outside the graph
        if (!ctx->capturing) ctx->gemv_ready_bytes = ctx->ws_bytes[WS_GEMV_PART];
    }
    const int64_t n_words = out * bits / 32;
    const dim3 grid(static_cast<unsigned>(sh.tiles), static_cast<unsigned>(sh.chunks));
    {
        ProfScope prof(ctx, "gemv_ic_tiles");
#define GV_GO(PB, LO, RANGES)                                                                                                    \
    do {                                                                                                                 \
        if (meta16)                                                                                                      \
            hipLaunchKernelGGL((gemv_ic_tiles<PB, true, LO, RANGES>), grid, dim3(64 * GV_WAVES), 0, ctx->stream, packed, scales, \
                               zeros, x, out, in, g, n_words, part, ticket, y);                                          \
        else                                                                                                             \
            hipLaunchKernelGGL((gemv_ic_tiles<PB, false, LO, RANGES>), grid, dim3(64 * GV_WAVES), 0, ctx->stream, packed, scales, \
                               zeros, x, out, in, g, n_words, part, ticket, y);                                          \
    } while (0)
        GV_PB(GV_GO)
#undef GV_GO
    }
    ADADIM_LAUNCH_CHECK(ctx, "gemv_ic_tiles");
    return ADADIM_OK;
}
