// Host check of csrc/gemv_plan.h: over many shapes, every quad of columns is taken by exactly one lane and step of a tile,
// ranges are those of 64-lane tiles (the order their sums are added up in), and no launch has fewer blocks
// than whole rounds of 64-lane tiles would give it.
#include "../../paper_2309_15531_amd/csrc/gemv_plan.h"

#include <cstdio>
#include <vector>

static long mistakes = 0;
static void check(bool ok, const char* what, int64_t out, int64_t in, int bits) {
    if (ok) return;
    if (++mistakes < 20) std::printf("%s: %lld x %lld, %d bits\n", what, (long long)out, (long long)in, bits);
}

template <int LO, bool RANGES>
static void columns(const GemvPlan& p, int64_t out, int64_t in, int bits) {
    constexpr uint32_t CL = 64 / LO;
    const uint32_t quads = static_cast<uint32_t>(in / 4);
    std::vector<int> taken(quads, 0);
    const uint32_t n = static_cast<uint32_t>(p.parts) * GV_WAVES, each = quads / n, more = quads % n;
    for (uint32_t y = 0; y < static_cast<uint32_t>(p.chunks); ++y)
        for (uint32_t w = 0; w < GV_WAVES; ++w) {
            uint32_t longest = 0;
            for (uint32_t cl = 0; cl < CL; ++cl) {
                const GemvColumns<LO, RANGES> c(in, static_cast<uint32_t>(p.chunks), y, w, cl);
                for (uint32_t s = 0; s < c.trips; ++s) {
                    const uint32_t q = c.quad(s);
                    check(q < quads, "a quad that does not exist", out, in, bits);
                    if (q < quads && c.has(s)) ++taken[q];
                    if (c.has(s) && s + 1 > longest) longest = s + 1;
                }
                if (RANGES) {                                 // range (y CL + cl) 8 + w of the 64-lane tile's parts * 8
                    const uint32_t r = (y * CL + cl) * GV_WAVES + w;
                    check(c.first == r * each + (r < more ? r : more) && c.count == each + (r < more ? 1 : 0) && c.trips >= c.count,
                          "another range than a 64-lane tile's", out, in, bits);
                    check(CL == 1 || c.count > 0, "an empty range", out, in, bits);
                }
            }
            const GemvColumns<LO, RANGES> c0(in, static_cast<uint32_t>(p.chunks), y, w, 0);
            check(longest == c0.trips, "a step without work", out, in, bits);
        }
    for (uint32_t q = 0; q < quads; ++q) check(taken[q] == 1, "a quad not taken exactly once", out, in, bits);
}

int main() {
    std::vector<int64_t> outs = {32, 64, 96, 256, 288, 512, 1024, 2048, 2080, 4096, 4128, 5632, 8192, 11008, 14336, 16352, 16384, 16416,
                                 22016, 28672, 32000, 32768, 49152, 65536, 67584, 88064, 128256, 131072, 133120, 151936, 174080, 262144,
                                 262176, 264192, 300032, 524288, 524320, 1048576, 1 << 24};
    std::vector<int64_t> ins = {4, 8, 32, 60, 64, 128, 252, 256, 260, 508, 512, 516, 768, 1024, 1028, 2048, 2572, 4096, 4100, 5120, 8192,
                                8196, 11008, 12288, 16384, 28672};
    long shapes = 0, ranges = 0;
    for (int64_t out : outs)
        for (int64_t in : ins)
            for (int c = 0; c < 12; ++c) {
                const int bits = 2 + c % 3, g = c / 3 & 1 ? 32 : 128;
                const bool meta16 = c >= 6;
                ++shapes;
                const GemvPlan p = gemv_plan(out, in, bits, g, meta16);
                const int64_t parts = gemv_round_parts(out, in), tiles64 = (out + 2047) / 2048;
                check(int64_t(p.tiles) * p.lo * 32 >= out && int64_t(p.tiles - 1) * p.lo * 32 < out, "tiles", out, in, bits);
                check(p.chunks >= 1 && p.parts <= parts, "more partial sums than whole rounds of 64-lane tiles", out, in, bits);
                check(p.chunks == 1 || p.tiles <= GV_SLOTS, "more counters than blocks in a round", out, in, bits);
                check(p.parts == (p.ranges ? p.chunks * (64 / p.lo) : p.chunks), "parts", out, in, bits);
                if (p.ranges) {
                    ++ranges;
                    check(p.parts == parts, "another number of parts than whole rounds have", out, in, bits);
                    check(p.lo == 64 || bits == 4, "a form that is not built", out, in, bits);
                }
                // the grid is at least nine tenths of what whole rounds of 64-lane tiles have
                // (two thirds of a round where short groups decide)
                if (out >= 2048)
                    check(10 * int64_t(p.tiles) * p.chunks >= 9 * tiles64 * parts || (g < 128 && 3 * p.tiles * p.chunks >= 2 * GV_SLOTS), "fewer blocks than whole rounds", out, in, bits);
                if (p.lo == 8) columns<8, false>(p, out, in, bits);
                else if (p.lo == 16) columns<16, false>(p, out, in, bits);
                else if (p.lo == 32 && p.ranges) columns<32, true>(p, out, in, bits);
                else if (p.lo == 32) columns<32, false>(p, out, in, bits);
                else columns<64, true>(p, out, in, bits);
            }
    std::printf("%ld shapes, %ld of them with a range per lane, %ld mistakes\n", shapes, ranges, mistakes);
    return mistakes ? 1 : 0;
}
