// Host check of csrc/factor_plan.h: follows the launches of a factor tile by tile.  In every launch a workgroup finds what it reads
// finished by earlier launches, nobody writes what another workgroup of the launch reads or writes, every element gets its products
// in order, and in the end every row of U has been written once from finished rows of the inverse.
//
// State per 64 x 64 tile.  A: columns of L subtracted so far; left of the panel, columns of the panel's own product made so far.
// M: above the diagonal L transposed (finished or not), in a panel's diagonal block its inverse (likewise), left of it how far
// L X has been added up.
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../paper_2309_15531_amd/csrc/factor_plan.h"

static long mistakes = 0;

struct Matrix {
    int64_t n, nt;
    std::vector<int> a, m, x, writer;                         // x: columns of a row panel's own product, in A
    std::vector<int> rows;                                    // how often a row of U was written
    std::vector<int> t;                                       // T's tiles: which level's product they hold
    std::vector<std::pair<int64_t, int>> reads, touched;      // (tile, workgroup) of this launch
    std::vector<std::pair<int*, int>> after;                  // states once it has ended
    long launches = 0;

    explicit Matrix(int64_t n) : n(n), nt((n + 63) / 64), a(nt * nt), m(nt * nt), x(nt * nt), writer(3 * nt * nt, -1), rows(n), t(64) {
        for (int64_t r = 0; r < nt; ++r)
            for (int64_t c = 0; c < r; ++c) m[r * nt + c] = static_cast<int>(c * 64);
    }
    void expect(bool ok, const char* what, int64_t i, int64_t j) {
        if (ok) return;
        if (++mistakes < 20) std::printf("%lld channels, launch %ld: %s (%lld, %lld)\n", (long long)n, launches, what, (long long)i, (long long)j);
    }
    void read(int64_t id, int wg) { reads.push_back({id, wg}); }
    void write(int64_t id, int wg, int* state, int value) {
        expect(writer[id] < 0, "written by two workgroups", id / nt, id % nt);
        writer[id] = wg;
        touched.push_back({id, wg});
        after.push_back({state, value});
    }
    int64_t A(int64_t r, int64_t c) const { return r * nt + c; }
    int64_t M(int64_t r, int64_t c) const { return nt * nt + r * nt + c; }
    int64_t T(int64_t i) const { return 2 * nt * nt + i; }
    void need_l(int64_t k, int64_t r, int wg) {               // L's block of row tile r, column tile k
        read(M(k, r), wg);
        expect(m[k * nt + r] == 1, "L is not there", r, k);
    }
    void need_inverse(int64_t r, int64_t c, int wg) {         // of a panel's diagonal block
        read(M(r, c), wg);
        expect(m[r * nt + c] == (r == c ? 1 : -1), "the diagonal block's inverse is not there", r, c);
    }
    void need_x(int64_t r, int64_t c, bool own, int wg) {     // a finished tile of the inverse
        if (own) return need_inverse(r, c, wg);
        read(A(r, c), wg);
        expect(x[r * nt + c] == static_cast<int>((r % 8 + 1) * 64), "a row of the inverse is not there", r, c);
    }
    void update(int64_t r, int64_t c, int64_t lo, int64_t hi, int wg) {       // A's tile gets the columns [lo, hi) of L
        read(A(r, c), wg);
        expect(a[r * nt + c] == lo, "an update out of order", r, c);
        for (int64_t k = lo / 64; k < hi / 64; ++k) {
            need_l(k, r, wg);
            need_l(k, c, wg);
        }
        write(A(r, c), wg, &a[r * nt + c], static_cast<int>(hi));
    }
    void diag(int64_t k, int wg) { write(M(k, k), wg, &m[k * nt + k], 1); }

    void job(const FactorJob& j, int tile, int wg) {
        const int64_t q = j.k0 / 64, end = std::min(nt, q + (j.w + 63) / 64);           // the panel's tiles [q, end)
        if (j.kind == FACTOR_T || j.kind == FACTOR_LEVEL) {
            const int64_t s = j.s / 64, pair = tile / (s * s), mt = tile / s % s, nn = tile % s, a0 = q + 2 * pair * s, b0 = a0 + s;
            expect(b0 < end, "a pair without rows", b0, end);
            if (b0 + mt >= end) return;
            const int64_t id = pair * s * s + mt * s + nn;
            if (j.kind == FACTOR_T) {
                for (int64_t k = nn; k < s; ++k) {
                    need_l(a0 + k, b0 + mt, wg);
                    need_inverse(a0 + k, a0 + nn, wg);
                }
                expect((id + 1) * 64 * 64 <= FACTOR_T_ELEMS, "T is too small", id, j.s);
                write(T(id), wg, &t[id], j.s + static_cast<int>(j.k0));
            } else {
                for (int64_t k = 0; k <= mt; ++k) {
                    need_inverse(b0 + mt, b0 + k, wg);
                    const int64_t from = pair * s * s + k * s + nn;
                    read(T(from), wg);
                    expect(t[from] == j.s + static_cast<int>(j.k0), "T is not there", from, j.s);
                }
                write(M(b0 + mt, a0 + nn), wg, &m[(b0 + mt) * nt + a0 + nn], -1);
            }
        } else if (j.kind == FACTOR_ROWS) {
            const int64_t cols = q, r = q + tile / cols, c = tile % cols, hi = std::min<int64_t>(j.hi, (r - q + 1) * 64);
            expect(r < end && j.lo < hi, "an empty product", r, c);
            expect(x[r * nt + c] == j.lo, "a panel's rows out of order", r, c);
            read(A(r, c), wg);
            for (int64_t k = j.lo / 64; k < hi / 64; ++k) {
                need_inverse(r, q + k, wg);
                read(M(q + k, c), wg);
                expect(m[(q + k) * nt + c] == j.k0, "L X is not complete", q + k, c);
            }
            write(A(r, c), wg, &x[r * nt + c], static_cast<int>(hi));
        } else if (j.kind == FACTOR_SPREAD) {
            const int64_t cols = end, r = end + tile / cols, c = tile % cols;
            expect(r < nt && j.w == FACTOR_NBO, "no rows below", r, c);
            const int64_t lo = std::max<int64_t>(j.k0 + j.lo, c * 64), hi = j.k0 + j.hi;
            if (lo >= hi) return;
            expect(m[r * nt + c] == lo, "L X out of order", r, c);
            for (int64_t k = lo / 64; k < hi / 64; ++k) {
                need_l(k, r, wg);
                need_x(k, c, c >= q, wg);
            }
            write(M(r, c), wg, &m[r * nt + c], static_cast<int>(hi));
        } else if (j.kind == FACTOR_FLIP) {
            const int64_t r = j.k0 + tile;
            expect(r < n && tile < j.w, "a row that does not exist", r, 0);
            for (int64_t c = 0; c <= r / 64; ++c) need_x(r / 64, c, c >= q, wg);
            if (r < n) after.push_back({&rows[r], rows[r] + 1});
        } else {
            int rt, ct;
            if (j.kind == FACTOR_NEXT) {
                rt = tile / j.s;
                ct = tile % j.s;
                if (ct > rt) return;
            } else {
                factor_behind(tile, rt, ct);
                expect(ct <= rt && ct >= 8, "above the diagonal", rt, ct);
            }
            const int64_t k1 = q + FACTOR_NBO / 64;
            expect(k1 + rt < nt, "a tile that does not exist", rt, ct);
            if (k1 + rt < nt) update(k1 + rt, k1 + ct, j.k0 + j.lo, j.k0 + j.hi, wg);
        }
    }

    void launch(const FactorLaunch& l) {
        ++launches;
        reads.clear();
        touched.clear();
        after.clear();
        const int64_t k = l.k0 / 64;
        int wg = 0;
        if (l.kind == FACTOR_DIAG) {
            read(A(k, k), wg);
            expect(a[k * nt + k] == l.k0, "the diagonal block is not up to date", k, k);
            diag(k, wg);
        } else if (l.kind == FACTOR_BELOW || l.kind == FACTOR_STEP) {
            const bool step = l.kind == FACTOR_STEP;
            expect(k + 1 + l.rows == nt, "rows", l.rows, nt);
            for (int rt = 0; rt < l.rows; ++rt)
                for (int ct = 0; ct < (step ? l.cols : 1); ++ct, ++wg) {
                    if (step && ct > rt) continue;
                    const int64_t r = k + 1 + rt, c = k + 1 + ct;
                    read(M(k, k), wg);
                    expect(m[k * nt + k] == 1, "the diagonal block is not factored", k, k);
                    for (int64_t i : {r, c}) {
                        if (!step && i == c) continue;
                        read(A(i, k), wg);
                        expect(a[i * nt + k] == l.k0, "the column is not up to date", i, k);
                    }
                    if (ct == 0) write(M(k, r), wg, &m[k * nt + r], 1);
                    if (!step) continue;
                    read(A(r, c), wg);
                    expect(a[r * nt + c] == l.k0, "a step out of order", r, c);
                    write(A(r, c), wg, &a[r * nt + c], static_cast<int>(l.k0 + 64));
                    if (wg == 0) diag(c, wg);
                }
        } else if (l.kind == FACTOR_UPDATE) {
            for (int rt = 0; rt < l.rows; ++rt)
                for (int ct = 0; ct < l.cols; ++ct, ++wg) {
                    if (ct > rt) continue;
                    update(l.k1 / 64 + rt, l.k1 / 64 + ct, l.k0, l.k0 + l.w, wg);
                    if (wg == 0) diag(l.k1 / 64, wg);
                }
        }
        expect(l.kind != FACTOR_JOBS || l.jobs.n > 0, "an empty launch", 0, 0);
        for (int i = 0; i < l.jobs.n; ++i) {
            expect(l.jobs.job[i].tiles > 0 && i < 7, "an empty job", i, l.jobs.job[i].kind);
            for (int tile = 0; tile < l.jobs.job[i].tiles; ++tile) job(l.jobs.job[i], l.jobs.job[i].from + tile, wg++);
        }
        for (auto& r : reads) expect(writer[r.first] < 0 || writer[r.first] == r.second, "read beside its write", r.first / nt, r.first % nt);
        for (auto& w : touched) writer[w.first] = -1;
        for (auto& s : after) *s.first = s.second;
    }
};

int main() {
    std::vector<int64_t> sizes;
    for (int64_t n = 1; n <= 2200; n = n < 1024 ? n + 61 : n + 23) sizes.push_back(n);
    for (int64_t n : {512, 576, 1024, 1025, 1088, 1089, 1536, 1537, 1600, 1601, 2048, 2049, 2100, 2560, 2561, 3000, 3333, 4096, 4097, 4608, 4609,
                      5120, 5121, 5600, 7168, 9001, 11008, 16400})
        sizes.push_back(n);
    long launches = 0;
    for (int64_t n : sizes) {
        Matrix mat(n);
        FactorPlan(n).run([&](const FactorLaunch& l) { mat.launch(l); });
        for (int64_t r = 0; r < n; ++r) mat.expect(mat.rows[r] == 1, "a row of U not written once", r, mat.rows[r]);
        launches += mat.launches;
    }
    // the widest factor: rows of workgroups, jobs included, that a grid can have
    for (int64_t n : {30000, 46340})
        FactorPlan(n).run([&](const FactorLaunch& l) {
            if (l.cols > 0 && l.rows + (l.jobs.tiles() + l.cols - 1) / l.cols > 52000) ++mistakes;
            ++launches;
        });
    // the order of the tiles behind, far beyond the sizes above
    int tile = 0;
    for (int r = 0; r < 1500; ++r)
        for (int c = 0; c <= r; ++c, ++tile) {
            int rt, ct;
            factor_behind(tile, rt, ct);
            if (rt != r + 8 || ct != c + 8) ++mistakes;
        }
    std::printf("%zu sizes, %ld launches, %ld mistakes\n", sizes.size(), launches, mistakes);
    return mistakes != 0;
}
