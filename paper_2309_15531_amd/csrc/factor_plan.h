// The launches of GPTQ's factor (gptq.hip) and what each carries.  Plain C++: tests/host/factor_plan_check.cpp follows them tile by
// tile on the CPU.
//
// The factorization is a chain of 64-wide steps inside 512-wide panels, a launch each, that leave most of the chip idle.  The update
// of the columns behind a panel, and the triangular inverse of the panels before, are cut into jobs, some tiles of 64 x 64 each,
// that travel in the steps' launches, behind the steps' workgroups: what a launch carries depends on earlier launches alone, and
// no other stream is needed.  With the update on a second stream and the inverse on a third, 4096 channels took 2210 us
// where the process used no others, 3100 to 3220 where two or three more were in use (there are four hardware queues, and
// two of the three streams shared one) and 3500 replayed from a recording; so 2220 in every case.  us, streams of their own and no
// others / so: 1100 587 / 529   2048 919 / 825   2900 1371 / 1335   5120 3405 / 3495   6144 4950 / 5410   8192 10030 / 10540   11008 21600 / 23070
// (8192 11900 beside two others; with the update alone on a second stream and the inverse at the end 4096 2607, 8192 10820, 11008 22500).
//
// A launch waits for its last tile, so tiles are short: the depth of 512 in two halves (a tile alone takes 17 us at a
// depth of 256 and 33 at 512, a step 19; 4096 2310 us so and 2490 in whole tiles, before launches were filled), unless a launch
// has so many that its end does not matter.  A tile more per compute unit makes a launch 10 us longer, so it is filled up to a
// multiple of 256 workgroups (4096 2240, 2290 without).
#pragma once

#include <algorithm>
#include <cstdint>

#if defined(__HIPCC__)
#define FACTOR_FN __host__ __device__ __forceinline__
#else
#define FACTOR_FN inline
#endif

constexpr int FACTOR_NB = 64;              // step, and edge of a tile
constexpr int FACTOR_NBO = 512;            // panel
constexpr int FACTOR_UNITS = 256;          // compute units
constexpr int64_t FACTOR_HALVES = 8192;    // tiles of a product beyond which they are not cut in two (11008 23410 cut, 23180 not)
// Channels up to which the next panel's columns get most of a panel's update ahead of the panel's end, us so / at its end: 1100 532 / 573,
// 2048 833 / 891, 4096 2251 / 2265, 5120 3577 / 3535, 8192 10770 / 10650
constexpr int64_t FACTOR_AHEAD = 4608;

// Elements of T: a level of size s has pairs of s x s, in a panel of 512 (256 squared at most) or in all of up to 1024 channels.
constexpr int64_t FACTOR_T_ELEMS = int64_t(FACTOR_NBO) * FACTOR_NBO;

enum FactorJobKind {
    FACTOR_T,          // T = C inv(A) of a doubling level of size s (a panel's diagonal block)
    FACTOR_LEVEL,      // M[B rows, A columns] = -inv(B) T of it
    FACTOR_ROWS,       // X's rows of the panel left of it, of the panel's 512 products per element those in [lo, hi)
    FACTOR_SPREAD,     // what the panel adds to the rows below, likewise
    FACTOR_FLIP,       // the panel's rows of U (a row per workgroup)
    FACTOR_NEXT,       // the panel's update of the next panel's columns (`s` tile columns), likewise
    FACTOR_BEHIND      // and of the columns behind those
};
struct FactorJob {
    int kind, from, tiles;                 // tiles [from, from + tiles) of it
    int w, s, lo, hi;                      // w: the panel's width
    int64_t k0;                            // the panel's first row
};
struct FactorJobs {
    int n = 0;
    FactorJob job[7];
    int tiles() const {
        int t = 0;
        for (int i = 0; i < n; ++i) t += job[i].tiles;
        return t;
    }
};

// tile row and column (from the next panel's first on) of tile `tile` of FACTOR_BEHIND: the lower triangle behind the next panel
FACTOR_FN void factor_behind(int tile, int& rt, int& ct) {
    int r = static_cast<int>((sqrtf(8.0f * static_cast<float>(tile) + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > tile) --r;
    while ((r + 1) * (r + 2) / 2 <= tile) ++r;
    rt = r + FACTOR_NBO / FACTOR_NB;
    ct = tile - r * (r + 1) / 2 + FACTOR_NBO / FACTOR_NB;
}

enum FactorLaunchKind {
    FACTOR_DIAG,       // factors and inverts the w wide diagonal block at k0
    FACTOR_STEP,       // the step at k0: L below the block there, cols x rows tiles of the panel behind it, the block at k0 + 64
    FACTOR_BELOW,      // L below the panel's last block, w wide, alone
    FACTOR_UPDATE,     // the update by L[., k0 .. k0 + w) of cols x rows tiles from k1 on, and the block at k1
    FACTOR_JOBS        // jobs alone
};
struct FactorLaunch {
    int kind;
    int64_t k0;
    int w;
    int64_t k1;
    int cols, rows;                        // tiles; those above the diagonal are none
    FactorJobs jobs;
};

// Calls launch(FactorLaunch) for the launches of an n wide factor, in order.
class FactorPlan {
    // tiles that several launches in a row carry: both halves of the depth one after the other, or whole
    struct Work {
        int kind;
        bool halves;
        int64_t panel = 0, tiles = 0, at = 0;                 // `at` of the tiles (of twice as many with halves) are given out
        int64_t left() const { return (halves ? 2 * tiles : tiles) - at; }
        void start(int64_t q, int64_t n) {
            panel = q;
            tiles = n;
            at = 0;
            if (kind != FACTOR_FLIP) halves = n <= FACTOR_HALVES;
        }
        // a launch's share, when `launches` (this one included) are to do the rest; never a tile's second half beside its first
        int64_t share(int64_t launches) const { return std::min((left() + launches - 1) / launches, tiles); }
        int64_t most() const { return std::min(left(), tiles); }
    };

    const int64_t n;
    const bool panels, ahead;              // more than two panels: jobs travel with the steps; see FACTOR_AHEAD
    const int64_t n_panels;                // of the inverse
    FactorJobs jobs;
    Work behind{FACTOR_BEHIND, true}, spread{FACTOR_SPREAD, true}, flip{FACTOR_FLIP, false};
    int64_t inverted = 0;                  // panel whose diagonal block is next
    int64_t size = FACTOR_NB;              // of the blocks that its next level pairs up
    bool has_t = false, half_rows = false; // the level's T is there; the first half of the panel's rows

    int64_t width(int64_t q) const { return panels ? std::min<int64_t>(n - q * FACTOR_NBO, FACTOR_NBO) : n; }
    int64_t tiles_below(int64_t q) const { return (n - std::min(n, (q + 1) * FACTOR_NBO) + FACTOR_NB - 1) / FACTOR_NB; }

    void add(int kind, int64_t q, int64_t s, int64_t from, int64_t tiles, int lo = 0, int hi = FACTOR_NBO) {
        if (tiles > 0)
            jobs.job[jobs.n++] = {kind, static_cast<int>(from), static_cast<int>(tiles), static_cast<int>(width(q)), static_cast<int>(s), lo,
                                  hi, q * FACTOR_NBO};
    }
    void give(Work& work, int64_t now) {
        if (work.halves) {
            const int64_t first = std::min(now, std::max<int64_t>(work.tiles - work.at, 0));
            add(work.kind, work.panel, 0, work.at, first, 0, FACTOR_NBO / 2);
            add(work.kind, work.panel, 0, work.at + first - work.tiles, now - first, FACTOR_NBO / 2, FACTOR_NBO);
        } else {
            add(work.kind, work.panel, 0, work.at, now);
        }
        work.at += now;
    }
    // The inverse's next link, panels < `done` being factored: a product of a doubling level; then the panel's rows, half by half, once all
    // that belongs to them has been added.  Whether it is the panel's rows.
    bool inverse(int64_t done) {
        if (inverted >= done) return false;
        const int64_t w = width(inverted);
        if (size < w) {
            const int64_t pairs = (w - size + 2 * size - 1) / (2 * size), across = size / FACTOR_NB;   // those with rows below the first block
            add(has_t ? FACTOR_LEVEL : FACTOR_T, inverted, size, 0, pairs * across * across);
            if (has_t) size *= 2;
            has_t = !has_t;
            return false;
        }
        if (!half_rows && spread.left() + flip.left() > 0) return false;
        const int64_t cols = inverted * (FACTOR_NBO / FACTOR_NB), rows = (w + FACTOR_NB - 1) / FACTOR_NB, top = std::min<int64_t>(rows, FACTOR_NBO / FACTOR_NB / 2);
        if (cols > 0 && !half_rows) {
            add(FACTOR_ROWS, inverted, 0, 0, cols * rows, 0, FACTOR_NBO / 2);
            half_rows = true;
            return true;
        }
        add(FACTOR_ROWS, inverted, 0, cols * top, cols * (rows - top), FACTOR_NBO / 2, FACTOR_NBO);      // (the upper rows have no second half)
        spread.start(inverted, inverted + 1 < n_panels ? (inverted + 1) * (FACTOR_NBO / FACTOR_NB) * tiles_below(inverted) : 0);
        flip.start(inverted, w);
        half_rows = false;
        ++inverted;
        size = FACTOR_NB;
        return cols > 0;
    }
    // The jobs of a launch of `own` workgroups beside those that `jobs` has, if the update behind a panel is to be done with
    // behind_in launches (0: none here) and what follows the inverse's rows with follow_in; rows: those rows are among the jobs.
    // (Beside their second half goes what needs the first half alone.)
    void shares(int64_t own, int64_t behind_in, int64_t follow_in, bool rows) {
        const bool spreads = !rows || spread.halves;
        int64_t now_b = behind_in > 0 ? behind.share(behind_in) : 0, now_s = spreads ? spread.share(follow_in) : 0;
        const int64_t now_f = rows ? 0 : flip.share(follow_in);
        int64_t room = FACTOR_UNITS - 1 - (own + jobs.tiles() + now_b + now_s + now_f + FACTOR_UNITS - 1) % FACTOR_UNITS;
        if (behind_in > 0) {
            const int64_t more = std::min(room, behind.most() - now_b);
            now_b += more;
            room -= more;
        }
        if (spreads) now_s += std::min(room, spread.most() - now_s);
        give(behind, now_b);
        give(spread, now_s);
        give(flip, now_f);
    }

public:
    explicit FactorPlan(int64_t n)
        : n(n), panels(n > 2 * FACTOR_NBO), ahead(n <= FACTOR_AHEAD), n_panels(panels ? (n + FACTOR_NBO - 1) / FACTOR_NBO : 1) {}

    template <typename F>
    void run(F launch) {
        constexpr int NB = FACTOR_NB, NBO = FACTOR_NBO;
        const int64_t last_slot = ahead ? 3 : 6;              // step by which the update behind the panel before is done
        bool diag = false;                                    // the block at the next k0 is factored
        for (int64_t K0 = 0; K0 < n; K0 += NBO) {
            const int64_t p = K0 / NBO, W = std::min<int64_t>(n - K0, NBO);
            const bool last = K0 + W == n;
            int64_t done = 0;                                 // of the panel's columns, how many the next panel's have had
            for (int64_t k0 = K0; k0 < K0 + W; k0 += NB) {
                const int w = static_cast<int>(std::min<int64_t>(n - k0, NB));
                if (!diag) launch(FactorLaunch{FACTOR_DIAG, k0, w, 0, 0, 0, {}});
                diag = false;
                const int64_t below = n - k0 - w;
                if (below == 0) break;
                const int rows = static_cast<int>((below + NB - 1) / NB), cols = static_cast<int>((K0 + W - k0 - w + NB - 1) / NB);
                if (cols == 0) {
                    launch(FactorLaunch{FACTOR_BELOW, k0, w, 0, 0, rows, {}});
                    continue;
                }
                jobs = {};
                if (panels) {
                    // a panel's rows come with its successor's last two steps, what follows them with the launches up to the next's
                    const int64_t slot = (k0 - K0) / NB;
                    const bool r = inverse(p);
                    if (ahead && !last) {
                        const int64_t across = std::min<int64_t>(tiles_below(p), NBO / NB), tiles = tiles_below(p) * across;
                        if (slot == 4) add(FACTOR_NEXT, p, across, 0, tiles / 2, 0, NBO / 2);
                        if (slot == 5) add(FACTOR_NEXT, p, across, tiles / 2, tiles - tiles / 2, 0, NBO / 2);
                        if (slot == 6) add(FACTOR_NEXT, p, across, 0, tiles, NBO / 2, 3 * NBO / 4);
                        done = 3 * NBO / 4;
                    }
                    shares(int64_t(cols) * rows, std::max<int64_t>(last_slot + 1 - slot, 1), slot < 5 ? 5 - slot : last ? 2 : 13 - slot, r);
                }
                launch(FactorLaunch{FACTOR_STEP, k0, NB, 0, cols, rows, jobs});
                diag = true;
            }
            if (last) break;
            // The panel's update of everything behind it: the next panel's own columns at once (the first tile's workgroup factors the
            // next diagonal block as well), which is all that its steps need; the columns behind those beside these steps.
            // Every element still receives the panels' updates in panel order.
            const int64_t rows = tiles_below(p), cols = panels ? std::min<int64_t>(rows, NBO / NB) : rows;
            jobs = {};
            if (panels) {
                behind.start(p, (rows - cols) * (rows - cols + 1) / 2);
                const bool r = inverse(p + 1);
                shares(cols * rows, last_slot + 2, 6, r);
            }
            launch(FactorLaunch{FACTOR_UPDATE, K0 + done, static_cast<int>(W - done), K0 + W, static_cast<int>(cols), static_cast<int>(rows), jobs});
            diag = true;
        }
        // what no step carried: for the last panel, and for one after which there were too few steps
        while (inverted < n_panels || spread.left() + flip.left() > 0) {
            jobs = {};
            const bool r = inverse(n_panels);
            shares(0, 0, 1, r);
            if (jobs.n > 0) launch(FactorLaunch{FACTOR_JOBS, 0, 0, 0, 0, 0, jobs});
        }
    }
};
