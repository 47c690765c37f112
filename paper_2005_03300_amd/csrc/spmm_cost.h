// What a sparse product costs in each of the schedules, estimated from how long the rows and the columns of the matrix are
// (host code without HIP).  The choice it makes is one of speed alone; every schedule computes every product.
//
// Two rates bound the gathers: what the L2s serve, and what they fetch (one 128-byte line per miss).  The misses follow from
// the distribution of the column lengths: the L2 of an XCD holds `C` lines, a line of rate r (its share of the accesses) is
// found there with probability 1 - exp(-r T), and T is such that the expected number of lines held is C (Che's
// approximation of an LRU cache); a line costs one miss in any case where it is touched at all.  That takes the vertices' order
// for random: a matrix of another keeps the schedule of the sizes (see even_rows, drawn_columns).  The constants were fitted to 600
// timed products (uniform, R-MAT and Chung-Lu graphs of 60 K to 4 M vertices, 26 to 490 entries per row, 16 to 128
// columns, 1 to 32 blocks, both schedules).  The cost of a partial row and the share of the blocks that an XCD walks were set again when the
// XCDs took stretches of the blocks (see chunk_group).  Estimates are within 12 % of the times in the root mean square, worse on
// R-MAT graphs and on narrow rows; a schedule other than that of the sizes is taken only where its estimated gain is beyond what they were
// found to be wrong by (must_save, narrow_panels, sweep_pays), at the price of gains below 10 to 20 %.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace gcn {

// How the rows of a matrix lie, taken from it when it is built (k_degrees, k_sample_columns): what tells an order of the vertices
// that groups like rows, or rows of like columns, from a random one.
struct RowOrder {
    static constexpr int GROUP = 64, LONG = 256;        // rows of a group; entries that a row counts with at the most
    static constexpr int WINDOWS = 16, GROUPS = 16, GROUP_ENTRIES = 2048, APART = 8, BITS = 18;
    double sum = 0, squares = 0;                        // of the groups' entries
    double distinct = 0;                                // columns among the WINDOW entries of a window, on average; 0: not sampled
    // A window is what the L2 of one XCD sees of a stretch of the matrix: every eighth group of 2048 entries (chunks go to
    // the XCDs in turn, four by four).
    static constexpr int WINDOW = GROUPS * GROUP_ENTRIES;
    static constexpr int64_t STRETCH = (int64_t)WINDOW * APART;
    // Every column of a window sets one bit of a table of 2^BITS (the factor is 2^32 over the golden ratio, which spreads numbers that
    // follow each other; applied twice, it leaves them as good as drawn); the number of columns follows from the number of bits.
#ifdef __HIPCC__
    __host__ __device__
#endif
    static uint32_t bit_of(uint32_t column) {
        uint32_t h = column * 0x9E3779B1u;
        h = (h ^ (h >> 15)) * 0x9E3779B1u;
        return h >> (32 - BITS);
    }
    static double distinct_of(const unsigned* ones) {
        double s = 0;
        const double m = (double)(1 << BITS);
        for (int w = 0; w < WINDOWS; ++w) s -= m * std::log(1.0 - std::min((double)ones[w], m - 1) / m);
        return s / WINDOWS;
    }
};

// How many rows (of a matrix, or of its transpose) have 2^b .. 2^(b+1) - 1 entries, and how many entries they hold.
struct Lengths {
    static constexpr int BINS = 32;
    int64_t rows[BINS] = {};
    int64_t entries[BINS] = {};
    int64_t total() const { int64_t t = 0; for (int64_t e : entries) t += e; return t; }
    int64_t count() const { int64_t t = 0; for (int64_t r : rows) t += r; return t; }
    // share of the entries that are in rows of eight times the mean and more
    double in_long_rows() const {
        const double all = std::max<double>(1.0, (double)total()), rows_all = (double)count();
        double in = 0;
        for (int b = 0; b < BINS; ++b)
            if (rows[b] > 0 && (double)entries[b] * rows_all > 8.0 * all * (double)rows[b]) in += (double)entries[b];
        return in / all;
    }
    // the rows of at least 2^b entries, or the others
    Lengths from(int b) const { Lengths l; for (int i = b; i < BINS; ++i) { l.rows[i] = rows[i]; l.entries[i] = entries[i]; } return l; }
    Lengths below(int b) const { Lengths l; for (int i = 0; i < b; ++i) { l.rows[i] = rows[i]; l.entries[i] = entries[i]; } return l; }
    // two of them at random on one line, three and four by doing it again: the lengths of the lines
    Lengths paired() const {
        Lengths l;
        double r[BINS] = {}, e[BINS] = {};
        const double all = std::max<double>(1.0, (double)count());
        for (int i = 0; i < BINS; ++i)
            for (int j = 0; rows[i] > 0 && j < BINS; ++j) {
                if (rows[j] <= 0) continue;
                const double n = 0.5 * (double)rows[i] * (double)rows[j] / all;
                const double d = (double)entries[i] / (double)rows[i] + (double)entries[j] / (double)rows[j];
                const int b = std::min(BINS - 1, (int)std::log2(d));
                r[b] += n;
                e[b] += n * d;
            }
        for (int i = 0; i < BINS; ++i)
            if (r[i] > 0) { l.rows[i] = std::max<int64_t>(1, (int64_t)(r[i] + 0.5)); l.entries[i] = std::max<int64_t>(1, (int64_t)(e[i] + 0.5)); }
        return l;
    }
    static Lengths equal(int64_t rows, int64_t entries) {        // all rows alike
        Lengths l;
        int b = 0;
        while (b < 31 && (2ll << b) * rows <= entries) ++b;
        l.rows[b] = rows;
        l.entries[b] = entries;
        return l;
    }
};

// The longest row that may go into a sweep copy of tasks of `rb` rows, whose places are counted in 32 bits: at worst every entry of a task
// makes a set of its own, and the last trip (at most 8 sets) is filled up.
inline int32_t longest_swept(int32_t rb, int32_t set) { return (int32_t)((INT32_MAX / set - 8) / rb); }

// How large the terms of a row are beside those of a longer one: values that are alike, whatever the row; 1 / sqrt(d_i d_j), which make the terms
// of a long row small, and 1 / d_i, which make them smaller.  UNKNOWN: the caller's values or row factors, which may be either.
enum class Terms { UNKNOWN, ALIKE, BY_BOTH, BY_ROW };

struct SpmmCost {
    int32_t f;                   // columns of the operand
    int cus;
    double xcds = 8, l2_bytes;

    int panel() const { return f <= 16 ? 16 : 32; }
    // Rows of 33 to 64 columns that are not whole 16-byte pieces are gathered in one panel, by as many lines as 4 f bytes at any
    // address touch on average; they share the lines at their ends.  (Taken for two panels of whole lines, they were given blocks
    // half as wide again as they should be: 41 columns, 6 M entries, 120 K vertices over two blocks 131 us, over three 122, estimated 132
    // and 122; 10 M, 150 K over four 220, over six 211.)
    bool ragged() const { return f % 4 != 0 && f > 32 && f <= 64; }
    int passes() const { return ragged() ? 1 : (f + 31) / 32; }
    double lines_per_row() const { return ragged() ? (4.0 * f + 124.0) / 128.0 : 1.0; }
    int rows_per_line() const { const int w = f < 32 ? f : 32; return w >= 17 ? 1 : 32 / (w < 1 ? 1 : w); }

    // The lines of X by the number of entries that select them.
    Lengths lines(const Lengths& cols) const {
        Lengths l = cols;
        for (int per = rows_per_line(); per > 1; per /= 2) l = l.paired();
        return l;
    }

    // Misses of one XCD: `accesses` to the lines that a `share` of the columns selects, which stay (`band`) or not.  A row of X
    // is `lines_each` lines.
    double misses(const Lengths& lines, double share, double accesses, bool band, double lines_each) const {
        const double all = std::max<double>(1.0, (double)lines.total()), c = l2_bytes * 0.835 / 128.0 / lines_each;        // the streams take some
        double n[Lengths::BINS], r[Lengths::BINS];
        int k = 0;
        for (int b = 0; b < Lengths::BINS; ++b)
            if (lines.rows[b] > 0) {
                n[k] = (double)lines.rows[b] * share;
                r[k++] = (double)lines.entries[b] / (double)lines.rows[b] / (all * share);
            }
        auto touched = [&](double t) { double s = 0; for (int i = 0; i < k; ++i) s += n[i] * (1.0 - std::exp(-r[i] * t)); return s; };
        const double once = touched(accesses);
        if (band || once <= c) return once;
        double lo = 0, hi = accesses;
        for (int it = 0; it < 40; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (touched(mid) < c) lo = mid; else hi = mid;
        }
        double s = 0;
        for (int i = 0; i < k; ++i) s += std::max(n[i] * (1.0 - std::exp(-r[i] * accesses)), n[i] * r[i] * accesses * std::exp(-r[i] * lo));
        return s;
    }

    // Share of the gathers over `blocks` column blocks that miss.
    double missed(const Lengths& lines, int blocks, double lines_each) const {
        const double each = std::max(1.0, blocks / xcds), all = std::max<double>(1.0, (double)lines.total());        // blocks that an XCD walks: each is in one of their L2s
        return misses(lines, 1.0 / blocks, all / xcds / each, false, lines_each) * xcds * each / all;
    }
    // Whether rows of 64 columns and more go over column blocks in panels of 32: half the panel misses less, but it takes two passes over the
    // entries.  Where a third of the gathers in panels of 64 would miss, and more, it took 0.65 to 1.00 of the time (430 products over 2 to
    // 16 blocks at 64 to 160 columns), where fewer would, 0.95 to 1.14; at 200 columns 0.92 to 1.06, at 67 and 101 1.02 to 1.25: not where
    // the pieces of a row start in the middle of half a line.
    bool narrow_panels(const Lengths& lines, int blocks) const {
        return f >= 64 && f % 16 == 0 && blocks >= 2 && missed(lines, blocks, 2.0) >= 0.34;
    }

    // Nonzero-split over `blocks` column blocks of the rows `rows` (microseconds); `lines` of the whole matrix.
    double split(const Lengths& rows, const Lengths& lines, int blocks) const {
        const double nnz = (double)rows.total(), w = lines_per_row(), fetched = nnz * passes() * w;
        const double m = nnz * missed(lines, blocks, ragged() ? f / 32.0 : 1.0) * passes() * w + nnz * passes() * 8 / 128;
        const bool narrow = f <= 16;
        const double served = fetched / (narrow ? 228e3 : 174e3), filled = m / (narrow ? 67.9e3 : 57.2e3);
        const double e = narrow ? 1.94 : 4.6;
        double t = std::pow(std::pow(served, e) + std::pow(filled, e), 1.0 / e) + 5.0;
        if (blocks > 1) {                        // partial rows: written, read, added
            double partial = 0;
            for (int b = 0; b < Lengths::BINS; ++b)
                if (rows.rows[b] > 0)
                    partial += (double)rows.rows[b] * blocks * (1.0 - std::pow(1.0 - 1.0 / blocks, (double)rows.entries[b] / (double)rows.rows[b]));
            t += partial * std::max(f, 16) * 4 * (narrow ? 0.47e-6 : 0.43e-6) + 7.6;
        }
        return t;
    }

    // How much less than the blocks of the sizes others have to cost: more than the estimates were found to be wrong by.  Of 2600 products of
    // 1 to 110 M entries (uniform, Chung-Lu, R-MAT; 100 K to 3.2 M vertices; 4 to 200 columns) timed over the blocks of the sizes and over more:
    // estimated at 0.82 to 0.94 of the cost, they took up to 1.35 of the time at 8 to 16 columns, up to 1.12 where most entries
    // are in long rows (R-MAT; such rows select cold columns one after the other), up to 1.08 at 17 to 32 columns over several
    // blocks instead of fewer, and 0.70 to 1.03 otherwise; estimated below the bound of their kind 0.45 to 1.03, but for a few of 8 columns up to 1.06.
    double must_save(const Lengths& rows, int usual, bool narrower) const {
        if (narrower) return 0.94;                              // (the sizes' panels of 64 take longer than the estimate has it)
        if (f <= 16) return usual >= 2 && f >= 8 ? 0.76 : 0.82;
        return rows.in_long_rows() > 0.42 || (usual >= 2 && (f <= 32 || f >= 64)) ? 0.82 : 0.94;
    }
    // Whether the sweep does.  4000 products timed in it and by the sizes: at 16 to 32 columns its estimate is 10 % too high beside the other's, but
    // for some 8 us of every product (estimated at 0.92 to 1.0 of the other's cost 246 products took 0.57 to 1.07 of the time, 1.02 and more those of
    // less than 120 us); wider ones took up to 1.00 below 0.92 and 1.28 beyond, those that are no whole lines 1.05 beyond 0.85, in two
    // panels (33 to 63 columns) beyond 0.75; of 8 to 15 columns 0.97 below 0.88, 1.12 beyond; below that 0.85 below 0.7, 1.07 beyond.  Nothing estimates the
    // hub schedule, which the sizes may choose below 32 columns where most entries are in rows of 64 and more: against it 0.92 of the
    // time below 0.75, at 16 columns and more 0.86 below 0.88, 1.15 and more beyond.
    bool sweep_pays(const Lengths& rows, double sweep, double split) const {
        if (f < 8) return sweep < 0.70 * split;
        if (f > 32) return sweep < (f < 64 ? 0.75 : (f % 32 == 0 ? 0.92 : 0.85)) * split;
        if (f < 32 && 2 * rows.from(6).total() > rows.total()) return sweep < (f < 16 ? 0.75 : 0.88) * split;
        return f < 16 ? sweep < 0.88 * split : sweep + 8.0 < 0.98 * split;
    }

    // The number of blocks that costs least, `usual` unless another is as much better as `must` says.  No fewer than usual: the
    // pieces of a sum would be longer, and its error larger.
    int best_blocks(const Lengths& rows, const Lengths& lines, int64_t ncols, int usual, double must, double* cost) const {
        static const int tried[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96};
        int best = usual;
        double least = split(rows, lines, usual);
        const double keep = least * must;
        for (int b : tried) {
            if (b == usual || (b > 1 && ncols / b < 2048) || b < usual) continue;
            const double t = split(rows, lines, b);
            if (t < keep && t < least) { least = t; best = b; }
        }
        *cost = least;
        return best;
    }

    // Places that the sweep stores per entry: a row takes one pair of steps per entry, so there is padding where a task's longest row has
    // more than its share.
    double padding(const Lengths& light, int64_t nrows, int32_t task_rows) const {
        int longest = 1;
        for (int b = 0; b < Lengths::BINS; ++b) if (light.rows[b] > 0) longest = b < 30 ? 2 << b : longest;
        const double places = 2.0 * (64 / (panel() / 4));
        return std::max(1.0, 0.55 * longest * places / (task_rows * (double)light.total() / (double)nrows));
    }

    // Column sweep: rows below 2^heavy entries in `tasks_per_cu` tasks of `task_rows` per compute unit, `parts` sums per row; the
    // others by the nonzero split (*heavy_blocks receives over how many blocks).
    double sweep(const Lengths& rows, const Lengths& lines, int64_t nrows, int64_t ncols, int heavy, int32_t task_rows, int tasks_per_cu,
                 int parts, int* heavy_blocks) const {
        const Lengths light = rows.below(heavy), rest = rows.from(heavy);
        const double nl = (double)light.total(), tasks = std::ceil((double)nrows / task_rows);
        const double launches = std::ceil(tasks / ((double)tasks_per_cu * cus));
        const int panels = (f + panel() - 1) / panel();
        *heavy_blocks = 1;
        if (nl <= 0) return 1e30;
        const double pad = padding(light, nrows, task_rows);
        const double fetched = nl * pad;
        const double m = launches * xcds * misses(lines, 1.0, nl / launches / xcds, true, 1.0) + fetched * 10 / 128;
        const double through = std::max(fetched / 130e3, m / 54e3);
        const double chain = launches * (fetched / tasks / (8.0 * 64 / (panel() / 4))) * 0.67;        // a trip takes 0.67 us
        double t = panels * (std::max(through, chain) + 4.0 * launches) + (parts - 1) * (double)nrows * f * 8 / 3.7e6;
        if (rest.total() > 0) {
            double h = 0;
            *heavy_blocks = best_blocks(rest, lines, ncols, 1, 0.94, &h);
            t += 1.41 * h + 8.0;
        }
        return t;
    }

    // ---- rounding errors ----
    // Every addition rounds in proportion to what has been added up; with terms alike in size the squares of these errors add up to
    // the number of terms in each sum so far, over all additions.  One chain of k terms:
    static double chain(double k) { return 0.5 * k * (k + 1); }
    // A row of `length` entries in the nonzero split over `blocks` blocks: chains that end where a lane group's slice of `slice`
    // entries does, wherever the row starts, joined in pairs; the blocks' sums are added one after another.
    static double split_error(double length, int slice, int blocks) {
        const double most = std::min(length, 2048.0);             // beyond that rows are alike: the slices bound the chains
        const double b = std::max(1.0, std::min((double)blocks, std::floor(most)));
        const int len = std::max(1, (int)(most / b + 0.5));
        double sum = 0, p[2048 / 32 + 2];
        const int step = slice / 16;
        for (int o = 0; o < slice; o += step) {
            int k = 0;
            for (int at = 0, end = slice - o; at < len; at = end, end += slice) p[k++] = std::min(end, len) - at;
            for (int i = 0; i < k; ++i) sum += chain(p[i]);
            for (; k > 1; k = (k + 1) / 2)
                for (int i = 0; i < k; i += 2) {
                    if (i + 1 < k) sum += p[i] + p[i + 1];
                    p[i / 2] = p[i] + (i + 1 < k ? p[i + 1] : 0);
                }
        }
        return b * sum / 16 + (most / b) * (0.5 * b * (b + 1) - 1.0);
    }
    // In the sweep: `parts` chains, of which each entry is in one or another, added one after another.
    static double sweep_error(double length, int parts) {
        const double p = parts, pieces = p * (1.0 - std::pow(1.0 - 1.0 / p, length));
        return 0.5 * (length * length / p + length * (1.0 - 1.0 / p) + length) +
               (pieces > 1 ? (length / pieces) * (0.5 * pieces * (pieces + 1) - 1.0) : 0.0);
    }
    // Over all rows, whose terms are in proportion to length^(power/2).  parts = 0: the nonzero split over `blocks`; otherwise rows below
    // 2^heavy entries in the sweep, the others over `blocks`.
    double error(const Lengths& rows, int blocks, int parts, int heavy, int power) const {
        double sum = 0;
        for (int b = 0; b < Lengths::BINS; ++b) {
            if (rows.rows[b] <= 0) continue;
            const double l = (double)rows.entries[b] / (double)rows.rows[b];
            sum += (double)rows.rows[b] * std::pow(l, power) *
                   (parts > 0 && b < heavy ? sweep_error(l, parts) : split_error(l, f <= 16 ? 32 : 64, blocks));
        }
        return sum;
    }
    // Whether sums in that schedule are as close to the exact ones as in the nonzero split over `usual` blocks.
    bool as_exact(const Lengths& rows, int usual, int blocks, int parts, int heavy, Terms terms) const {
        // One chain per row grows with the squares of the lengths, which are taken to be alike within a factor of two: measured up to 2 %
        // further off than the nonzero split where this had them equal (uniform rows of 12, Chung-Lu rows of 20 times 1 / d_i, at 32 columns).
        const double most = parts == 1 ? 0.9 : 1.0;
        auto holds = [&](int power) { return error(rows, blocks, parts, heavy, power) <= most * error(rows, usual, 0, heavy, power); };
        switch (terms) {
            case Terms::ALIKE: return holds(0);
            case Terms::BY_BOTH: return holds(-1);
            case Terms::BY_ROW: return holds(-2);
            default: return holds(0) && holds(-2);
        }
    }
};

// Whether nothing in a matrix tells its order of vertices from a random one, so that the estimates hold.
//
// Rows: groups of 64 of them differ in their entries (counted up to 256 per row) no more than rows drawn at random make them: the
// squares of the differences add up to those of the single rows.  Four times that, or a tenth of the mean, is let pass.  (The same of
// the transpose's rows tells the columns'.)
inline bool even_rows(const Lengths& rows, int64_t nrows, const RowOrder& order) {
    const double mean = order.sum / std::max<double>(1.0, (double)nrows);
    double alone = std::max(0.0, (double)nrows - (double)rows.count()) * mean * mean;
    for (int b = 0; b < Lengths::BINS; ++b)
        if (rows.rows[b] > 0) {
            const double d = std::min((double)rows.entries[b] / (double)rows.rows[b], (double)RowOrder::LONG) - mean;
            alone += (double)rows.rows[b] * d * d;
        }
    const double full = std::floor((double)nrows / RowOrder::GROUP) * RowOrder::GROUP, left = (double)nrows - full;
    const double even = mean * mean * (full * RowOrder::GROUP + left * left);
    return order.squares - even <= 4.0 * alone + 0.01 * even;
}
// Columns: the entries that an XCD meets one after the other select as many different ones as draws by the columns' lengths would.
// Measured 0.98 to 1.02 of that on 95 graphs renamed at random; with vertices numbered along a band of 20 K, in 64 communities with half
// of the edges inside, or with distances by a power law 0.53 to 0.89, and there the schedule that the estimates give
// took up to 1.8 times as long as the one of the sizes.
inline bool drawn_columns(const Lengths& cols, const RowOrder& order) {
    const double all = std::max<double>(1.0, (double)cols.total());
    double drawn = 0;
    for (int b = 0; b < Lengths::BINS; ++b)
        if (cols.rows[b] > 0)
            drawn += (double)cols.rows[b] * (1.0 - std::exp(-(double)RowOrder::WINDOW * ((double)cols.entries[b] / (double)cols.rows[b]) / all));
    return order.distinct > 0 && order.distinct >= 0.94 * drawn;
}

// The schedule of a product whose order of additions is free (see SpmmOpt::any_schedule).
struct SpmmPlan {
    int32_t f = 0;
    Terms terms = Terms::UNKNOWN;
    bool sweep = false;
    int32_t blocks = 1;          // column blocks: of the matrix, or of the sweep's long rows
    bool narrow = false;         // these in panels of 32
    int32_t parts = 1, heavy = 0;// sweep: sums per row, long-row threshold
    int32_t usual = 1;           // blocks by the sizes alone
    double padding = 1;          // sweep: places per entry, estimated
    bool by_sizes() const { return !sweep && blocks == usual; }
    void give_way() { sweep = narrow = false; blocks = usual; }
};

// Runs a product (`run` leaves the plan it followed, if any, in its argument).  The stored order of a planned schedule is there for
// speed: where there is no memory for it, this and later products of that width take the schedule of the sizes.
template <class Run>
int run_or_by_sizes(int out_of_memory, const Run& run) {
    SpmmPlan* plan = nullptr;
    const int rc = run(&plan);
    if (rc != out_of_memory || !plan || plan->by_sizes()) return rc;
    plan->give_way();
    plan = nullptr;
    return run(&plan);
}

}  // namespace gcn
