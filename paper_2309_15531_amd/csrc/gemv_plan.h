// Launch shape of the de-quantizing matrix-vector product (gemv_ic.hip): lanes of a wave along the outputs, output tiles,
// blocks per tile, partial sums per output, and which columns a lane takes.  Plain C++: tests/host/gemv_plan_check.cpp runs it
// on the CPU.
#pragma once

#include <algorithm>
#include <cstdint>

#if defined(__HIPCC__)
#define GEMV_FN __host__ __device__ __forceinline__
#else
#define GEMV_FN inline
#endif

constexpr int GV_WAVES = 8;
constexpr int GV_SLOTS = 256;              // blocks per round: one per compute unit (two would fit, and are 5 % slower)
constexpr int GV_MIN_COLS = 32;            // columns a range of the wide form has at least

struct GemvPlan {
    int lo;                                // lanes along the outputs: 8, 16, 32 or 64
    int tiles, chunks;                     // the grid: output tiles of 32 lo, blocks per tile
    int parts;                             // partial sums per output that the blocks of a tile leave
    bool ranges;                           // every column lane has a range of columns of its own, else they take turns
};

// Partial sums per output of 64-lane tiles whose blocks fill whole rounds, every wave keeping GV_MIN_COLS columns.
inline int64_t gemv_round_parts(int64_t out, int64_t in, int64_t* by_slots = nullptr) {
    const int64_t tiles = (out + 2047) / 2048, rounds = (tiles + GV_SLOTS - 1) / GV_SLOTS;
    const int64_t fill = std::max<int64_t>(1, rounds * GV_SLOTS / tiles), most = std::max<int64_t>(1, in / (GV_WAVES * GV_MIN_COLS));
    if (by_slots) *by_slots = fill;
    return std::min(fill, most);
}

// Wide layers (outputs enough that tiles of 64 lanes fill the rounds with GV_MIN_COLS columns per wave) have
// gemv_round_parts parts of 8 waves each, whose sums are added up in the same order by the two forms with ranges:
//   ranges, 64 lanes: a block per part;
//   ranges, 32 lanes: two parts per block, one for each column lane (an even number of parts): as many blocks, half as many
//       outputs to add up in each;
//   turns, 32 lanes: the two column lanes take turns, which reads the groups' parameters in twice as long pieces but adds up
//       in another order (the results move by rounding).
// Odd parts take 64 lanes, even ones 32; turns only where ranges would lose against 64 lanes in two launches, the form
// before: with an even number where parameters or codes come in short pieces (groups shorter than 128, columns that do not
// start on a 128-byte line, less than four bits), with an odd number where the parameters are a
// sixteenth of a byte or more per weight, if the tiles of 32 lanes fill two thirds of a round (they have half a part less: at
// 151936 outputs a third of the compute units has no block), or where more than eight parts are many to add up and those
// tiles fill seven eighths of a round.
// Everything smaller: tiles as narrow as it takes to have enough blocks; column lanes take turns.  Tiles are cut into several
// blocks up to one round of them, with at least two steps per wave: with fewer the partial sums cost more than the shorter
// wait for the loads saves.
//
// Measured back to back, weights beyond the caches, us.  Small, LO = 8 / 16, and 64 in two launches:
//   4096 x 4096, 4 bits     8.2   8.3  19.8        4096 x 4096, 3 bits     8.8   8.2  20.1
//   1024 x 8192, 4 bits     7.6   8.6  19.8        4096 x 11008, 4 bits   12.1  12.5  31.3
//   11008 x 4096, 4 bits   11.1  11.0  21.5        8192 x 28672, 4 bits   30.5  28.6  50.6
// Even parts, ranges / turns / 64 lanes in two launches (w: group words; groups of 128, the last two 32):
//   16384 x 8192, 4 bits   20.7  20.3  24.7        49152 x 12288, 4 bits  64.0  61.6  68.1
//   49152 x 12288, 4, w    56.7  59.1  59.0        65536 x 8192, 4 bits   52.2  53.4  59.0
//   49152 x 12288, 3 bits  56.6  50.6  55.5        16384 x 8192, 3, w     19.3  18.5  18.5
//   32000 x 8192, 3 bits   30.9  27.4  28.6        128256 x 4096, 3 bits  52.0  44.6  47.9
//   32032 x 5120, 4 bits   42.5  30.5  40.1        50272 x 8192, 4 bits  109.0  75.6  90.8
// Odd parts, ranges / turns / 64 lanes in two launches (groups of 128, the third line 32,
// the last 13 and 17 parts):
//   88064 x 4096, 4 bits   41.0  44.1  45.8        151552 x 4096, 4 bits  64.0  76.9  72.0
//   88064 x 4096, 3 bits   34.8  37.9  35.7        151552 x 4096, 3 bits  56.1  66.0  57.4
//   88064 x 4096, 4 bits   74.2  64.0  78.0        45056 x 8192, 3 bits   64.5  50.0  62.8
//   38912 x 4096, 2 bits   19.4  17.4  18.5        29696 x 7336, 4 bits   29.7  25.4  31.5
inline GemvPlan gemv_plan(int64_t out, int64_t in, int bits, int64_t g, bool meta16) {
    GemvPlan s;
    int64_t fill = 0;
    const int64_t parts = gemv_round_parts(out, in, &fill);
    if (out >= 16384 && parts == fill) {
        const int tiles32 = static_cast<int>((out + 1023) / 1024), turns = std::max(1, GV_SLOTS / tiles32);
        if (parts % 2 == 0) s.ranges = bits == 4 && g >= 128 && out % 256 == 0;
        else s.ranges = !(((meta16 ? 2 : 5) * 16 >= g && 3 * tiles32 * turns >= 2 * GV_SLOTS) || (parts > 8 && 8 * tiles32 * turns >= 7 * GV_SLOTS));
        s.lo = s.ranges && parts % 2 != 0 ? 64 : 32;
        s.tiles = s.lo == 64 ? static_cast<int>((out + 2047) / 2048) : tiles32;
        s.chunks = static_cast<int>(s.ranges ? parts * s.lo / 64 : turns);
        s.parts = static_cast<int>(s.ranges ? parts : turns);
        return s;
    }
    s.ranges = false;
    s.lo = out > 4096 || (bits < 4 && out > 2048) ? 16 : 8;
    s.tiles = static_cast<int>((out + s.lo * 32 - 1) / (s.lo * 32));
    const int64_t steps = (in / 4 + 64 / s.lo - 1) / (64 / s.lo);
    s.chunks = static_cast<int>(std::max<int64_t>(1, std::min({int64_t(GV_SLOTS / s.tiles), steps / (2 * GV_WAVES), parts})));
    s.parts = s.chunks;
    return s;
}

// The columns of one lane, in steps of a quad of four.  RANGES: every column lane of every wave has a range of its own, the
// in/4 quads dealt evenly to blocks * CL * 8 ranges, the first `quads % ranges` taking one more; lane cl of wave w of block y
// has range (y CL + cl) 8 + w.  Else a wave has a range of steps of CL quads, one for each column lane.  `trips` is the
// same in the whole wave; a lane has nothing to do in a step that `has` denies (the quad it is given then exists all the
// same).
template <int LO, bool RANGES>
struct GemvColumns {
    static constexpr uint32_t CL = 64 / LO;                   // column lanes
    uint32_t first, count, trips, quads, lane;
    GEMV_FN GemvColumns(int64_t in, uint32_t blocks, uint32_t block, uint32_t wave, uint32_t cl)
        : quads(static_cast<uint32_t>(in >> 2)), lane(cl) {
        const uint32_t n = blocks * GV_WAVES * (RANGES ? CL : 1), all = RANGES ? quads : (quads + CL - 1) / CL;
        const uint32_t each = all / n, more = all - each * n;
        const uint32_t wave0 = block * (RANGES ? CL : 1) * GV_WAVES + wave;             // the wave's first range
        const uint32_t mine = wave0 + (RANGES ? cl * GV_WAVES : 0);
        first = mine * each + (mine < more ? mine : more);
        count = each + (mine < more ? 1u : 0u);
        trips = each + (wave0 < more ? 1u : 0u);
    }
    GEMV_FN bool has(uint32_t s) const { return CL == 1 || (RANGES ? s < count : (first + s) * CL + lane < quads); }
    GEMV_FN uint32_t quad(uint32_t s) const {
        if (CL == 1) return first + s;                                                   // (s < trips)
        if (RANGES) return first + (s < count ? s : count - 1);                          // (no range is empty)
        const uint32_t q = (first + s) * CL + lane;
        return q < quads ? q : quads - 1;
    }
};
