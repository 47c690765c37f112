"""Host-side parts of the library that need no GPU, compiled by themselves with the host compiler."""
import os
import subprocess
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_03300_amd", "csrc")


def run_cpp(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(textwrap.dedent(body))
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)


def test_the_largest_request_is_never_followed_by_a_smaller_one(tmp_path):
    """Two threads ask for different sizes; the one with the smaller size is held inside its request until the other one
    has made its own (or is found to wait for it).  What was asked for last must be the larger one, and be remembered."""
    r = run_cpp(tmp_path, """
        #include <chrono>
        #include <cstdio>
        #include <thread>
        #include "largest_asked.h"
        int main() {
            gcn::LargestAsked kept;
            std::atomic<size_t> setting{0};
            std::atomic<bool> small_inside{false}, large_done{false};
            std::thread small([&] {
                kept.reach(50, [&](size_t v) {
                    small_inside = true;
                    for (int i = 0; i < 300 && !large_done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
                    setting = v;
                    return true;
                });
            });
            std::thread large([&] {
                while (!small_inside) std::this_thread::yield();
                kept.reach(100, [&](size_t v) { setting = v; return true; });
                large_done = true;
            });
            small.join();
            large.join();
            std::printf("%zu ", (size_t)setting);
            int asked_again = 0;
            kept.reach(100, [&](size_t) { ++asked_again; return true; });
            kept.reach(70, [&](size_t) { ++asked_again; return true; });
            kept.reach(120, [&](size_t) { ++asked_again; return false; });      // refused: asked again next time
            kept.reach(120, [&](size_t v) { setting = v; ++asked_again; return true; });
            std::printf("%zu %d", (size_t)setting, asked_again);
        }
    """)
    assert r.returncode == 0 and r.stdout == "100 120 2", (r.returncode, r.stdout, r.stderr)


def test_estimated_costs_choose_as_timed(tmp_path):
    """The cost of a sparse product by schedule: on matrices whose products were timed in every schedule the one chosen is within 10 %
    of the fastest; degenerate matrices give finite numbers and no division by zero."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "spmm_cost.h"
        using namespace gcn;
        static Lengths uniform(int64_t n, int64_t mean) { return Lengths::equal(n, n * mean); }
        int main() {
            struct { int64_t n, mean; int f; double split, sweep; } timed[] = {      // microseconds; best number of blocks
                {500000, 41, 16, 271, 164}, {500000, 41, 32, 404, 234}, {1000000, 61, 16, 874, 475}, {1000000, 61, 64, 2465, 1352},
                {2000000, 41, 16, 1622, 715}, {4000000, 26, 64, 4404, 3793}, {200000, 201, 16, 229, 465}, {200000, 201, 64, 660, 946}};
            for (auto& t : timed) {
                const SpmmCost c{t.f, 256, 8.0, 4.0 * (1 << 20)};
                const Lengths rows = uniform(t.n, t.mean), l = c.lines(rows);
                double split = 0;
                int hb = 0;
                const int b = c.best_blocks(rows, l, t.n, 1, c.must_save(rows, 1, false), &split);
                const double sweep = c.sweep(rows, l, t.n, t.n, 8, t.f <= 16 ? 511 : 255, 5, 1, &hb);
                const bool right = (sweep < split) == (t.sweep < t.split) || std::fabs(t.sweep / t.split - 1) < 0.1;
                std::printf("%d%d%d ", (int)right, (int)(split > 0.7 * t.split && split < 1.4 * t.split), (int)(sweep > 0.7 * t.sweep && sweep < 1.4 * t.sweep));
                (void)b;
            }
            int hb = 0;
            double x = 0;
            const SpmmCost c{4, 256, 8.0, 4.0 * (1 << 20)};
            Lengths none, one = uniform(1, 1), longest;
            longest.rows[30] = 1;
            longest.entries[30] = 1ll << 30;
            for (const Lengths& l : {one, longest})
                for (int64_t n : {1ll, 1ll << 31}) {
                    c.best_blocks(l, c.lines(l), n, 1, 0.9, &x);
                    if (!std::isfinite(x) || !std::isfinite(c.sweep(l, c.lines(l), n, n, 8, 511, 5, 3, &hb)) || hb < 1) std::printf("bad ");
                }
            c.best_blocks(none, c.lines(none), 1, 1, 0.9, &x);
            std::printf(std::isfinite(x) ? "ok" : "bad");
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["111"] * 8 + ["ok"], (r.returncode, r.stdout, r.stderr)


def test_schedules_of_skewed_matrices_are_not_changed_for_worse(tmp_path):
    """Renamed power-law graphs whose products were timed by the sizes and in another schedule (column blocks, narrower panels, sweep): where the other one
    took longer, by 7 to 35 %, the product keeps the schedule of the sizes; where it took at least a quarter less, it does not."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "spmm_cost.h"
        using namespace gcn;
        int main() {
            struct { int f; int64_t n; int usual, other; double sizes, us; int64_t rows[20], entries[20]; } timed[] = {      // other: blocks, or -1 for the sweep
                {16, 675186, 6, 12, 749, 826,      // Chung-Lu 2.3
                 {0, 0, 0, 0, 5076, 300760, 223083, 87671, 35080, 14174, 5639, 2267, 894, 352, 131, 52, 7},
                 {0, 0, 0, 0, 147971, 14702678, 19408359, 15313048, 12269416, 9929442, 7904851, 6343942, 5001566, 3946723, 2932200, 2319702, 509646}},
                {64, 347117, 6, 8, 1468, 1069,      // Chung-Lu 3.0
                 {0, 0, 0, 0, 0, 322, 199977, 110806, 27155, 6669, 1664, 409, 102, 13},
                 {0, 0, 0, 0, 0, 19565, 19857316, 18824723, 9249552, 4549048, 2271359, 1116087, 554376, 118617}},
                {64, 369072, 7, 7, 1587, 1166,      // Chung-Lu 3.0
                 {0, 0, 0, 0, 0, 93, 196082, 130646, 31842, 7842, 1946, 481, 121, 19},
                 {0, 0, 0, 0, 0, 5668, 20028805, 22195493, 10851746, 5352967, 2659340, 1310320, 656469, 179984}},
                {64, 101762, 7, 7, 251, 284,      // R-MAT
                 {7676, 10417, 11314, 12516, 16930, 4606, 16669, 9929, 2388, 6076, 2289, 118, 680, 136, 17, 1},
                 {7676, 25454, 60455, 129704, 414250, 187899, 1348980, 2291067, 687169, 4293136, 4398163, 260204, 3330949, 1511809, 377989, 38586}},
                {128, 112570, 6, 6, 458, 522,      // R-MAT
                 {11161, 13637, 15287, 12088, 19584, 8365, 10915, 11874, 323, 6102, 2380, 21, 679, 136, 17, 1},
                 {11161, 33023, 82466, 124766, 431292, 464708, 788156, 2358949, 99228, 3614149, 3911260, 48254, 2886741, 1342726, 346141, 36510}},
                {8, 2766711, 1, 24, 530, 715,      // Chung-Lu 2.1
                 {125892, 731512, 1122483, 478072, 175632, 73464, 32579, 14747, 6726, 3083, 1402, 628, 281, 125, 54, 24, 7},
                 {125892, 1879539, 5784293, 4958765, 3760640, 3194307, 2857279, 2598683, 2373193, 2177934, 1979146, 1768976, 1580826, 1404822, 1210214, 1075229, 558663}},
                {16, 486654, 1, 8, 404, 299,      // Chung-Lu 3.0
                 {0, 0, 0, 360, 124497, 272324, 68017, 16182, 3994, 979, 240, 61},
                 {0, 0, 0, 5126, 3346797, 11616681, 5750578, 2746033, 1358920, 667279, 327698, 165476}},
                {32, 790548, 1, 3, 413, 458,      // R-MAT
                 {220198, 153017, 121044, 75091, 85773, 60181, 15780, 37546, 2350, 13341, 4840, 36, 1140, 190, 19, 1, 1},
                 {220198, 363200, 638895, 807943, 1752886, 3195822, 1137653, 6606832, 1117669, 7320595, 7884400, 78700, 5423713, 2463061, 617404, 32821, 73202}},
                {48, 405282, 1, 8, 1386, 944,      // Chung-Lu 2.5
                 {0, 0, 0, 12, 28709, 227614, 97852, 33325, 11565, 4039, 1431, 496, 173, 57, 9},
                 {0, 0, 0, 167, 809622, 10260311, 8438447, 5776163, 4014265, 2803026, 1987807, 1381704, 968640, 637471, 164437}},
                {64, 331220, 1, 8, 923, 689,      // Chung-Lu 3.0
                 {0, 0, 0, 0, 1702, 182144, 112089, 26647, 6507, 1619, 401, 98, 13},
                 {0, 0, 0, 0, 50030, 9036513, 9477344, 4532026, 2215101, 1102454, 546834, 267456, 58958}},
                {64, 509906, 1, 3, 710, 798,      // R-MAT
                 {111245, 91201, 71171, 65455, 63101, 14307, 49625, 13636, 13501, 11628, 0, 3876, 969, 165, 6, 19, 1},
                 {111245, 218307, 372568, 676847, 1582929, 512648, 4115681, 3315687, 3622033, 9054439, 0, 8869414, 6141567, 2666992, 98656, 708151, 77100}},
                {16, 643482, 1, -1, 245, 160,      // Chung-Lu 3.0
                 {4, 222, 16081, 271423, 275724, 61617, 14026, 3323, 815, 199, 48},
                 {4, 629, 102062, 3290609, 5752465, 2579136, 1184486, 565616, 277686, 135157, 62718}},
                {64, 1193664, 1, -1, 2891, 1851,      // Chung-Lu 3.0
                 {0, 0, 0, 49, 136075, 761458, 224815, 53861, 13118, 3244, 798, 201, 45},
                 {0, 0, 0, 703, 3806637, 33505945, 19002534, 9145006, 4468460, 2217367, 1090641, 550250, 238637}}};
            for (auto& t : timed) {
                const SpmmCost c{t.f, 256, 8.0, 4.0 * (1 << 20)};
                Lengths rows;
                for (int b = 0; b < 20; ++b) { rows.rows[b] = t.rows[b]; rows.entries[b] = t.entries[b]; }
                const Lengths l = c.lines(rows);
                double split = 0;
                int hb = 0, parts = 1;
                const bool narrow = c.narrow_panels(l, t.usual);
                const int b = c.best_blocks(rows, l, t.n, t.usual, c.must_save(rows, t.usual, narrow), &split);
                while (parts <= 8 && !c.as_exact(rows, t.usual, 1, parts, 8, Terms::BY_BOTH)) ++parts;
                const double sweep = parts > 8 ? 1e30 : c.sweep(rows, l, t.n, t.n, 8, t.f <= 16 ? 511 : 255, 5, parts, &hb);
                const bool other = narrow || b != t.usual || c.sweep_pays(rows, sweep, split);
                std::printf("%d ", other == (t.us < t.sizes));
            }
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["1"] * 13, (r.returncode, r.stdout, r.stderr)


def test_estimated_costs_of_ragged_rows(tmp_path):
    """Blocks for rows of 33 to 64 columns that are no whole 16-byte pieces, on uniform matrices timed over 1 to 8 blocks: what is
    chosen takes no more than 5 % longer than the fastest; the widths beside that range are estimated as before."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "spmm_cost.h"
        using namespace gcn;
        int main() {
            struct { int64_t n, mean; int f, usual; double us[9]; } timed[] = {       // microseconds by number of blocks
                {150000, 67, 41, 2, {0, 344, 299, 252, 220, 0, 211, 0, 227}}, {150000, 67, 47, 2, {0, 380, 340, 292, 256, 0, 240, 0, 253}},
                {100000, 81, 41, 3, {0, 243, 188, 154, 152, 0, 148, 0, 158}}, {100000, 81, 47, 3, {0, 274, 219, 176, 168, 0, 163, 0, 169}}};
            for (auto& t : timed) {
                const SpmmCost c{t.f, 256, 8.0, 4.0 * (1 << 20)};
                const Lengths rows = Lengths::equal(t.n, t.n * t.mean);
                double cost = 0, least = 1e30;
                const int b = c.best_blocks(rows, c.lines(rows), t.n, t.usual, c.must_save(rows, t.usual, false), &cost);
                for (double us : t.us) if (us > 0) least = std::min(least, us);
                std::printf("%d ", b <= 8 && t.us[b] > 0 && t.us[b] <= 1.05 * least);
            }
            for (int f : {31, 32, 33, 36, 63, 64, 65, 127}) {
                const SpmmCost c{f, 256, 8.0, 4.0 * (1 << 20)};
                std::printf("%d%d ", c.passes(), c.lines_per_row() == 1.0);
            }
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["1"] * 4 + ["11", "11", "10", "21", "10", "21", "31", "41"], (r.returncode, r.stdout, r.stderr)


def test_places_of_a_sweep_task_fit_32_bits(tmp_path):
    """A task whose rows are as long as the sweep takes them, every entry in a set of its own and the last trip filled up, has fewer than
    2^31 places, at the task heights in use and at the least and the greatest; no such row is left out without need."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "spmm_cost.h"
        using namespace gcn;
        int main() {
            for (int rb : {1, 255, 511, 4096})
                for (int set : {16, 32}) {
                    const int64_t trip = 4 * set, longest = longest_swept(rb, set);
                    const int64_t places = (rb * longest * set + trip - 1) / trip * trip, more = rb * (longest + 1) * set + 8 * set;
                    std::printf("%d ", longest > 1024 && places <= INT32_MAX && more > INT32_MAX);
                }
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["1"] * 8, (r.returncode, r.stdout, r.stderr)


def test_a_planned_schedule_without_memory_gives_way_to_the_one_by_sizes(tmp_path):
    """A product whose planned stored order cannot be allocated runs by sizes, then and later; any other error, and no memory for the
    schedule of the sizes itself, is the caller's."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "spmm_cost.h"
        using namespace gcn;
        int main() {
            const int OK = 0, OOM = -4, HIP = -6;
            for (int copy : {OK, OOM, HIP})
                for (int plain : {OK, OOM})
                    for (int kind = 0; kind < 4; ++kind) {          // no plan, sweep, other blocks, the blocks of the sizes
                        SpmmPlan kept;
                        kept.usual = 2;
                        kept.sweep = kind == 1;
                        kept.blocks = kind == 2 ? 8 : (kind == 1 ? 1 : 2);
                        int runs = 0;
                        auto product = [&](SpmmPlan** plan) {
                            ++runs;
                            if (kind) *plan = &kept;
                            return kind && !kept.by_sizes() ? copy : plain;
                        };
                        const bool planned = kind == 1 || kind == 2;
                        const int first = run_or_by_sizes(OOM, product), one = runs;
                        const int again = run_or_by_sizes(OOM, product), two = runs - one;
                        const int want = planned && copy != OOM ? copy : plain;
                        const bool gave_way = planned && copy == OOM;
                        if (first != want || again != want || one != 1 + gave_way || two != 1 || kept.by_sizes() != (!planned || gave_way))
                            std::printf("%d/%d/%d: %d %d %d %d ", copy, plain, kind, first, again, one, two);
                    }
            std::printf("done");
        }
    """)
    assert r.returncode == 0 and r.stdout == "done", (r.returncode, r.stdout, r.stderr)


def test_an_order_of_the_vertices_that_is_not_random_is_told(tmp_path):
    """Rows of all lengths and columns drawn at random pass; rows sorted by length, denser and sparser halves, and windows that select fewer
    columns than draws would do not.  Rows that are all alike, empty ones and single ones divide by nothing."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <random>
        #include <vector>
        #include "spmm_cost.h"
        using namespace gcn;
        static Lengths lengths(const std::vector<int>& d) {
            Lengths l;
            for (int x : d) if (x > 0) { const int b = (int)std::log2((double)x); l.rows[b]++; l.entries[b] += x; }
            return l;
        }
        static RowOrder order(const std::vector<int>& d) {
            RowOrder o;
            for (size_t i = 0; i < d.size(); i += RowOrder::GROUP) {
                double g = 0;
                for (size_t k = i; k < d.size() && k < i + RowOrder::GROUP; ++k) g += std::min(d[k], (int)RowOrder::LONG);
                o.sum += g;
                o.squares += g * g;
            }
            return o;
        }
        int main() {
            std::mt19937 gen(7);
            std::uniform_real_distribution<double> u(0, 1);
            for (int n : {1, 63, 64, 65, 5000, 200000}) {
                std::vector<int> poisson(n), power(n), alike(n, 40), none(n, 0), halves(n);
                std::poisson_distribution<int> p(30), dense(60), thin(15);
                for (int i = 0; i < n; ++i) {
                    poisson[i] = p(gen);
                    power[i] = std::min(20000, (int)(4 * std::pow(u(gen), -0.75)));
                    halves[i] = i < n / 2 ? dense(gen) : thin(gen);
                }
                std::vector<int> sorted = power;
                std::sort(sorted.begin(), sorted.end());
                for (auto* d : {&poisson, &power, &alike, &none}) std::printf("%d", even_rows(lengths(*d), n, order(*d)));
                if (n >= 5000) std::printf("%d%d", even_rows(lengths(sorted), n, order(sorted)), even_rows(lengths(halves), n, order(halves)));
                std::printf(" ");
            }
            // windows of as many entries as drawn, by the table of bits; then of 0.85 times as many
            const int n = 150000;
            std::vector<int> d(n);
            for (int& x : d) x = 1 + (int)(8 * std::pow(u(gen), -0.7));
            std::vector<int> pick;
            for (int i = 0; i < n; ++i) for (int k = 0; k < d[i]; ++k) pick.push_back(i);
            for (double keep : {1.0, 0.85}) {
                unsigned ones[RowOrder::WINDOWS] = {};
                for (unsigned& o : ones) {
                    std::vector<bool> bit(1 << RowOrder::BITS);
                    for (int k = 0; k < RowOrder::WINDOW * keep; ++k) bit[RowOrder::bit_of((uint32_t)pick[(size_t)(u(gen) * pick.size())])] = true;
                    for (bool b : bit) o += b;
                }
                RowOrder o;
                std::printf("%d", drawn_columns(lengths(d), o));             // not sampled
                o.distinct = RowOrder::distinct_of(ones);
                std::printf("%d ", drawn_columns(lengths(d), o));
            }
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["1111"] * 4 + ["111100"] * 2 + ["01", "00"], (r.returncode, r.stdout, r.stderr)


def test_estimated_rounding_errors(tmp_path):
    """The squared error of a row's sum in either schedule, in units of one rounding of one term, against sums added up in single precision in that
    very order; and the number of sums per row that follows is no less exact than the nonzero split for rows of 12 to 200 entries."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <random>
        #include <vector>
        #include "spmm_cost.h"
        using namespace gcn;
        int main() {
            std::mt19937 gen(11);
            std::uniform_real_distribution<double> value(-1, 1), u(0, 1);
            const int rows = 6000;
            double unit = 0;
            for (int length : {16, 20, 41, 100})
                for (int parts = 0; parts <= 3; ++parts) {
                    double square = 0;
                    for (int r = 0; r < rows; ++r) {
                        std::vector<std::vector<double>> piece(1);
                        double exact = 0;
                        const int offset = (int)(u(gen) * 32);
                        std::vector<int> in(length);
                        for (int& p : in) p = (int)(u(gen) * std::max(1, parts));
                        std::sort(in.begin(), in.end());
                        for (int k = 0; k < length; ++k) {
                            if (k > 0 && (parts ? in[k] != in[k - 1] : (k + offset) % 32 == 0)) piece.emplace_back();
                            piece.back().push_back(value(gen) * 0.3);
                            exact += piece.back().back();
                        }
                        std::vector<float> sum;
                        for (auto& p : piece) {
                            float s = 0;
                            for (double x : p) s = (float)((double)s + x);
                            sum.push_back(s);
                        }
                        if (parts) for (size_t i = 1; i < sum.size(); ++i) sum[0] = sum[0] + sum[i];
                        else
                            while (sum.size() > 1) {
                                std::vector<float> next;
                                for (size_t i = 0; i < sum.size(); i += 2) next.push_back(i + 1 < sum.size() ? sum[i] + sum[i + 1] : sum[i]);
                                sum = next;
                            }
                        square += (sum[0] - exact) * (sum[0] - exact) / rows;
                    }
                    const double model = parts ? SpmmCost::sweep_error(length, parts) : SpmmCost::split_error(length, 32, 1);
                    if (unit == 0) unit = square / model;
                    const double ratio = std::sqrt(square / (model * unit));
                    if (ratio < 0.9 || ratio > 1.1) std::printf("length %d parts %d: %.2f ", length, parts, ratio);
                }
            for (int mean : {12, 16, 20, 21, 25, 41, 61, 100, 200})
                for (int f : {16, 32}) {
                    const SpmmCost c{f, 256, 8.0, 4.0 * (1 << 20)};
                    const Lengths l = Lengths::equal(1 << 20, (int64_t)mean << 20);
                    for (bool normalised : {false, true}) {
                        int parts = 1;
                        while (parts < 20 && !c.as_exact(l, 1, 1, parts, 8, normalised ? Terms::BY_BOTH : Terms::UNKNOWN)) ++parts;
                        if (SpmmCost::sweep_error(mean, parts) > SpmmCost::split_error(mean, f <= 16 ? 32 : 64, 1) || parts < 2 || parts > 8)
                            std::printf("mean %d f %d: %d sums ", mean, f, parts);
                    }
                    if (!c.as_exact(l, 4, 4, 0, 8, Terms::BY_BOTH) || c.as_exact(l, 4, 2, 0, 8, Terms::BY_BOTH)) std::printf("blocks %d %d ", mean, f);
                }
            std::printf("done");
        }
    """)
    assert r.returncode == 0 and r.stdout == "done", (r.returncode, r.stdout, r.stderr)


def test_a_kernel_copies_only_on_the_matrix_own_gpu(tmp_path):
    """An export by a kernel: the matrix, the destination and the stream on the current GPU, the whole range in one allocation and a multiple
    of 16 bytes; a matrix of another GPU, whose memory a kernel there may not reach, goes the runtime's way."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <initializer_list>
        #include "copy_rule.h"
        using namespace gcn;
        int main() {
            const MemoryOf here{true, 0, 4096, 1024}, there{true, 1, 4096, 1024}, host{false, -1, 0, 0};
            std::printf("%d%d%d%d ", kernel_copies(0, 0, 0, here, 4096, 1024), kernel_copies(1, 1, 1, there, 4096, 1024), kernel_copies(0, 0, 0, here, 4112, 1008),
                        kernel_copies(0, 0, 0, here, 5120, 0));
            int other = 0;                                    // any of the four on another GPU
            for (int m = 0; m < 2; ++m)
                for (int c = 0; c < 2; ++c)
                    for (int s = -1; s < 2; ++s)
                        for (const MemoryOf& of : {here, there})
                            if (!(m == c && c == s && s == of.gpu)) other += kernel_copies(m, c, s, of, 4096, 64);
            std::printf("%d ", other);
            std::printf("%d%d%d%d%d%d", kernel_copies(0, 0, 0, host, 4096, 64), kernel_copies(0, 0, 0, here, 4100, 64), kernel_copies(0, 0, 0, here, 4096, 1025),
                        kernel_copies(0, 0, 0, here, 4112, 1024), kernel_copies(0, 0, 0, here, 4080, 16), kernel_copies(0, 0, 0, here, 4112, ~(size_t)0));
        }
    """)
    assert r.returncode == 0 and r.stdout == "1111 0 000000", (r.returncode, r.stdout, r.stderr)


def test_wavefronts_of_dense_products_as_timed(tmp_path):
    """Four wavefronts or eight, at sizes on both sides of the rule: what took less, and where the rule takes the slower by no more than 16 %."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <initializer_list>
        #include "launch_rules.h"
        int main() {
            struct { int rows, panels, k; double eight, four; } timed[] = {      // microseconds
                {5000, 1, 128, 5.33, 4.41}, {16384, 1, 128, 5.49, 4.55}, {14400, 1, 256, 7.29, 6.17}, {14400, 1, 300, 17.4, 15.5}, {16384, 1, 16, 4.72, 4.24},
                {20000, 1, 256, 10.73, 11.97}, {32768, 1, 256, 18.2, 20.7}, {20000, 1, 400, 24.4, 35.3}, {5000, 1, 500, 15.9, 14.2}, {10000, 1, 640, 13.88, 11.18},
                {16384, 1, 602, 21.4, 23.6}, {5000, 1, 602, 18.2, 16.4}, {9000, 2, 602, 27.5, 52.1}, {3000, 2, 1200, 21.5, 26.0}, {8192, 1, 1200, 26.8, 30.0},
                {18000, 2, 100, 13.3, 12.4}, {23000, 2, 160, 17.6, 15.7}, {20000, 2, 16, 6.23, 5.88}, {10000, 2, 128, 9.80, 10.29}, {14000, 2, 200, 14.5, 15.9},
                {5000, 2, 300, 16.6, 14.3}, {5000, 4, 128, 9.05, 9.85}, {10000, 4, 100, 13.5, 12.8}, {12288, 4, 128, 14.8, 13.8}, {10000, 4, 200, 22.1, 27.1},
                {14000, 4, 100, 14.9, 16.2}, {3000, 1, 1900, 30.39, 28.08}, {3000, 2, 1900, 31.7, 43.47}, {5000, 1, 800, 23.49, 21.53}, {26000, 4, 100, 21.7, 24.1}};
            struct { int rows, panels, k; double eight, four; } slower[] = {     // the largest of what the rule gives away
                {10000, 1, 500, 16.9, 18.8}, {14336, 1, 416, 12.94, 14.66}, {2000, 8, 1000, 27.85, 24.52}};
            for (auto& t : timed) std::printf("%d", (int)((gcn::tall_waves((t.rows + 15) / 16, t.panels, t.k, 256) == 4) == (t.four < t.eight)));
            for (auto& t : slower) {
                const double took = gcn::tall_waves((t.rows + 15) / 16, t.panels, t.k, 256) == 4 ? t.four : t.eight;
                std::printf("%d", (int)(took <= 1.16 * (t.four < t.eight ? t.four : t.eight)));
            }
            for (int cus : {1, 8, 64, 256, 304}) std::printf(" %d", gcn::tall_waves(8 * cus + 1, 1, 16, cus));
        }
    """)
    assert r.returncode == 0 and r.stdout == "1" * 33 + " 8" * 5, (r.returncode, r.stdout, r.stderr)


def test_empty_rows_go_with_the_chunks_only_where_that_was_faster(tmp_path):
    """Products of random matrices timed with a launch that zeroes the rows without entries and with a share of them for every chunk: the rule
    shares where that took less, and not where it took longer, by up to a half; all rows are in some chunk's share."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "launch_rules.h"
        using gcn::share_of_empty_rows;
        int main() {
            struct { long long n, n_empty, chunks; int lpr, vec, f; double launch, share; } timed[] = {      // microseconds
                {3000, 136, 20, 16, 4, 64, 1, 1}, {3000, 1807, 13, 4, 4, 16, 12.9, 12.0}, {20000, 12080, 86, 8, 4, 128, 21.9, 20.0}, {20000, 12080, 86, 8, 4, 64, 18.7, 17.9},
                {3000, 2096, 8, 8, 4, 64, 18.1, 19.2}, {3000, 2096, 8, 32, 1, 31, 35.4, 42.4}, {150001, 119922, 506, 32, 1, 31, 41.9, 45.9}, {400000, 238680, 1755, 32, 1, 31, 57.2, 53.1},
                {20000, 18576, 86, 32, 1, 31, 25.1, 30.9}, {60000, 48000, 199, 32, 1, 31, 35.2, 43.1}, {1000000, 300000, 6285, 32, 1, 31, 161.8, 161.9}, {400000, 238680, 1755, 64, 1, 41, 62.8, 63.4},
                {400000, 197550, 2195, 64, 1, 41, 70.4, 74.3}, {1000000, 696210, 5045, 64, 1, 41, 160.5, 149.6}, {60000, 47959, 199, 8, 4, 128, 27.5, 25.1}, {1000000, 696210, 5045, 8, 4, 64, 165.1, 149.6},
                {1000000, 300000, 7661, 8, 4, 300, 1551, 1701}, {1000000, 800000, 3356, 8, 4, 300, 904, 1294}, {1000000, 800000, 3356, 8, 4, 100, 334, 461}, {2000000, 1200000, 8754, 8, 4, 36, 350, 396},
                {400000, 280000, 2014, 8, 4, 36, 73.1, 77.5}, {150001, 105000, 757, 8, 4, 200, 110.5, 116.3}, {3000, 600, 27, 8, 4, 300, 18.7, 16.6}, {20000, 10000, 108, 8, 4, 100, 21.6, 20.2},
                {1000000, 300000, 6285, 8, 4, 128, 355.8, 339.9}, {1000000, 800000, 3356, 8, 4, 160, 330.9, 283.1}, {1000000, 800000, 3356, 8, 4, 20, 72.9, 71.6},
                {60000, 48750, 178, 4, 4, 16, 12.7, 13.9}, {3000000, 2250001, 1500, 4, 4, 16, 1, 2}};                     // more of them than entries
            for (auto& t : timed) {
                const int share = share_of_empty_rows(t.n, t.n_empty, t.chunks, 512, t.lpr, t.vec, t.f, t.f, 1 << 20);
                if (share && (share > 512 || share * t.chunks < t.n_empty)) std::printf("lost ");
                std::printf("%d", (int)((share > 0) == (t.share <= t.launch * 1.001)));
            }
            const long long n = 1000000, e = 800000;
            std::printf(" %d%d%d%d%d", share_of_empty_rows(n, 0, 10, 512, 8, 4, 16, 16, 0), share_of_empty_rows(n, 5, 0, 512, 8, 4, 16, 16, 0),
                        share_of_empty_rows(n, e, 3356, 512, 8, 4, 128, 132, 1 << 20), share_of_empty_rows(n, e, 3356, 512, 8, 4, 128, 128, 16),
                        share_of_empty_rows(n, 10, 10, 512, 8, 4, 16, 17, 4));
        }
    """)
    assert r.returncode == 0 and r.stdout == "1" * 29 + " 00001", (r.returncode, r.stdout, r.stderr)


def test_a_padded_copy_of_short_rows_is_made_where_its_kernel_was_faster(tmp_path):
    """Matrices of 60 K short rows and fewer timed with the kernel of equal pitch and with the nonzero split."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "launch_rules.h"
        int main() {
            struct { int rows, pitch; long long nnz; int rows_of_16; double padded, split; } timed[] = {      // microseconds
                {60000, 64, 750000, 17700, 15.7, 13.1}, {60000, 64, 1272000, 30100, 18.0, 15.1}, {65500, 64, 831850, 19300, 16.7, 13.5}, {52000, 64, 655200, 15300, 13.8, 13.0},
                {44000, 64, 550000, 13000, 12.7, 13.6}, {32000, 64, 403200, 9400, 9.9, 12.3}, {60000, 64, 300060, 1, 10.4, 13.1}, {60000, 64, 3840000, 60000, 26.3, 37.3},
                {60000, 64, 1920000, 45000, 20.7, 21.2}, {60000, 20, 1020000, 60000, 10.8, 11.8}, {60000, 4, 180000, 0, 4.9, 6.7}, {1, 4, 1, 0, 1, 2}};
            for (auto& t : timed) std::printf("%d", (int)(gcn::short_copy_pays(t.rows, t.pitch, t.nnz, t.rows_of_16) == (t.padded < t.split)));
        }
    """)
    assert r.returncode == 0 and r.stdout == "1" * 12, (r.returncode, r.stdout, r.stderr)


def test_wavefronts_that_add_up_partial_results(tmp_path):
    """One to a partial result: none without one, none more than 16."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <initializer_list>
        #include "launch_rules.h"
        int main() {
            for (long long parts : {0ll, 1ll, 2ll, 15ll, 16ll, 17ll, 1ll << 40}) std::printf("%d ", gcn::sum_waves(parts));
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "1 1 2 15 16 16 16".split(), (r.returncode, r.stdout, r.stderr)


def test_scratch_of_calls_that_overlap(tmp_path):
    """A buffer belongs to one call at a time, those of a stream stay on it, and all memory is given back once.  Two threads each write their
    name into what they are given and find it there when they are done."""
    r = run_cpp(tmp_path, """
        #include <atomic>
        #include <cstdio>
        #include <cstdlib>
        #include <set>
        #include <thread>
        #include "scratch_pool.h"
        int main() {
            gcn::ScratchPool pool;
            std::set<void*> live;
            int fails = 0;
            auto alloc = [&](void** p, size_t bytes) { *p = std::malloc(bytes); live.insert(*p); return 0; };
            int s1 = 0, s2 = 0;
            void *a, *b, *c, *d, *e;
            pool.take(0, &s1, 100, &a, alloc);
            pool.take(0, &s1, 100, &b, alloc);              // the first one is out
            pool.take(0, &s2, 100, &c, alloc);
            pool.take(1, &s1, 100, &d, alloc);
            std::printf("%d ", (int)live.size());
            pool.give(a);
            pool.take(0, &s1, 125, &e, alloc);              // 100 and a quarter
            std::printf("%d ", (int)(e == a));
            pool.give(e);
            pool.give(b);
            pool.take(0, &s1, 1000, &e, alloc);             // one of the two is replaced, and kept
            pool.take(0, &s1, 10, &a, alloc);
            std::printf("%d %d ", (int)live.size(), (int)(a != e));
            void* none = &s1;
            const int rc = pool.take(0, &s1, 5000, &none, [&](void**, size_t) { ++fails; return -4; });
            std::printf("%d %d %d ", rc, fails, (int)(none == &s1));
            pool.give(a);
            pool.give(e);
            pool.take(0, &s1, 600, &b, alloc);
            pool.take(0, &s1, 60, &a, alloc);
            std::printf("%d%d ", (int)(b == e), (int)live.size());
            pool.give(a); pool.give(b); pool.give(c); pool.give(d);
            std::atomic<int> mixed{0};
            auto work = [&](int name) {
                for (int i = 0; i < 20000; ++i) {
                    void* p;
                    pool.take(0, &s1, 64, &p, [](void** q, size_t bytes) { *q = std::malloc(bytes); return 0; });
                    volatile int* const at = (volatile int*)p;
                    for (int k = 0; k < 16; ++k) at[k] = name;
                    for (int k = 0; k < 16; ++k) mixed += at[k] != name;
                    pool.give(p);
                }
            };
            std::thread t(work, 1), u(work, 2);
            t.join();
            u.join();
            int freed = 0;
            pool.clear([&](void* p) { freed += (int)live.erase(p); std::free(p); });
            pool.clear([&](void*) { freed += 100; });
            std::printf("%d %d %d", (int)mixed, freed, (int)live.size());
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "4 1 5 1 -4 1 1 15 0 5 0".split(), (r.returncode, r.stdout, r.stderr)


def test_room_for_the_end_of_an_epoch(tmp_path):
    """Partial results lie in memory that is idle from the loss on, apart from each other; wherever the plain shares fit the scaled operand's region and the scratch (or the
    first T) in turn, there is room; and gradients over few rows get theirs: the first layer's at any number of rows, also with a last share that is not whole."""
    r = run_cpp(tmp_path, """
        #include <algorithm>
        #include <cmath>
        #include <cstdio>
        #include <random>
        #include "epoch_layout.h"
        using namespace gcn;
        struct Range { size_t from, to; };
        static bool in_order(const EpochLayout& lay, int64_t n, int L, const int32_t* dims, bool vf, bool p0, bool fuse) {      // the plain shares, first fit
            size_t left[2] = {0, 0};
            if (L >= 8) return false;
            if (!vf) left[0] = lay.scratch - lay.XS;
            else if (p0 || (lay.order[0] == GCN_ORDER_GEMM_FIRST && L >= 2)) left[0] = lay.G[0] - lay.T[0];
            if (!fuse) left[1] = lay.total - lay.scratch;
            bool some = left[0] || left[1];
            auto take = [&](size_t b) {
                b = round256(b);
                for (size_t& l : left) if (b <= l) { l -= b; return true; }
                return false;
            };
            bool all = fuse || take((size_t)std::min<int64_t>((n + 3) / 4, 2048) * 8);
            for (int l = fuse ? L - 2 : L - 1; l >= 0 && all; --l) all = take(tn_shape(dims[l], dims[l + 1], n, false).scratch_bytes);
            return all && some;
        }
        int main() {
            std::mt19937 rng(5);
            auto pick = [&](int a, int b) { return a + (int)(rng() % (unsigned)(b - a + 1)); };
            const int widths[] = {1, 3, 4, 8, 12, 16, 16, 16, 20, 32, 48, 63, 64, 64, 100, 300};
            int lost = 0, bad = 0, few = 0, could = 0;
            for (int i = 0; i < 200000; ++i) {
                int64_t n = (int64_t)std::exp(pick(0, 1100) / 100.0);
                if (pick(0, 2) == 0) n = (n / 64 + 1) * 64;
                if (pick(0, 9) == 0) n *= 50;
                const int L = pick(1, 8);
                int32_t dims[9];
                for (int l = 0; l <= L; ++l) dims[l] = pick(0, 9) ? widths[pick(0, 15)] : pick(1, 300);
                const int order = pick(0, 4) % 3;
                const bool vf = pick(0, 2) == 0, p0 = pick(0, 3) == 0;
                const EpochLayout lay = epoch_layout(n, L, dims, order);
                const int mode = pick(0, 3) % 3;
                const bool fuse = mode && !(lay.order[L - 1] == GCN_ORDER_GEMM_FIRST && !(L == 1 && p0)) && fused_last_supported(dims[L - 1], dims[L]);
                const bool keep = fuse && mode == 2;
                const EpochRoom room = epoch_room(lay, n, L, dims, vf, p0, fuse, keep);
                if (!room.any) { lost += in_order(lay, n, L, dims, vf, p0, fuse); continue; }
                std::vector<Range> idle, used;
                if (!vf) idle.push_back({lay.XS, fuse ? lay.scratch : lay.total});
                else if (!fuse) idle.push_back({lay.scratch, lay.total});
                if (!(fuse && L == 1)) for (int l = 0; l < L; ++l)
                    if ((l == 0 && p0) || lay.order[l] == GCN_ORDER_GEMM_FIRST) idle.push_back({lay.T[l], lay.G[l]});
                if (fuse && !keep) idle.push_back({lay.T[L - 1], lay.S});
                auto use = [&](size_t at, size_t bytes) {
                    const Range u = {at, at + bytes};
                    bool inside = false;
                    for (const Range& r : idle) inside = inside || (r.from <= u.from && u.to <= r.to);
                    for (const Range& r : used) if (u.from < r.to && r.from < u.to) inside = false;
                    if (!inside || at % 256) ++bad;
                    used.push_back(u);
                };
                if (!fuse) {
                    use(room.loss, loss_part_bytes(n, dims[L]));
                    if (!p0 && room.loss >= lay.T[L - 1] && room.loss < lay.G[L - 1]) ++bad;           // (the loss may come from the product that reads it)
                }
                for (int l = fuse ? L - 2 : L - 1; l >= 0; --l) {
                    use(room.grad[l], tn_shape(dims[l], dims[l + 1], n, room.few[l]).scratch_bytes);
                    if (room.few[l] && !few_rows(dims[l], dims[l + 1], n)) ++bad;
                    could += few_rows(dims[l], dims[l + 1], n);
                    few += room.few[l];
                }
            }
            std::printf("%d %d %d ", lost, bad, (int)(few > 10000 && few > 0.95 * could));
            const int32_t a[] = {16, 64, 8}, b[] = {8, 64, 4}, g[] = {4, 10}, h[] = {5, 16, 32, 8}, c[] = {64, 16, 8}, d[] = {64, 16, 41}, e[] = {64, 16}, f[] = {63, 16, 16, 12};
            int none = 0, plain = 0;
            for (int64_t n = 64; n <= 16384; n += n < 5000 ? 1 : 61) {
                auto room = [&](int L, const int32_t* dims, bool fuse) { return epoch_room(epoch_layout(n, L, dims, 0), n, L, dims, false, false, fuse, false); };
                const EpochRoom r[] = {room(2, c, false), room(2, d, true), room(2, d, false), room(1, e, false), room(3, f, false), room(1, g, false), room(3, h, false)};
                none += !room(2, a, false).any + !room(2, b, false).any;
                for (const EpochRoom& x : r) { none += !x.any; plain += !x.few[0]; }
                none += (size_t)epoch_layout(n, 2, c, 0).total - epoch_layout(n, 2, c, 0).XS < tn_shape(64, 16, n, true).scratch_bytes;     // without room: one after another
            }
            std::printf("%d %d", none, plain);
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "0 0 1 0 0".split(), (r.returncode, r.stdout, r.stderr)


def test_products_by_themselves_are_cut_for_few_rows_where_that_is_faster(tmp_path):
    """Shares of 64 rows of a product by itself: up to 20 K rows, 12 K with more than 32 columns on a side, and never where an epoch's gradient would not have them; beyond, the
    longer shares of other products."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "epoch_layout.h"
        using namespace gcn;
        int main() {
            int wrong = 0;
            for (int M = 1; M <= 80; ++M)
                for (int N = 1; N <= 80; ++N)
                    for (int64_t K : {1, 63, 64, 1000, 12000, 12001, 16384, 20000, 20001, 32768, 40000}) {
                        const int wide = M > N ? M : N, narrow = M > N ? N : M;
                        const bool want = K >= 64 && narrow <= 16 && (wide <= 32 ? K <= 20000 : wide <= 64 && K <= 12000);
                        wrong += few_rows_alone(M, N, K) != want || (want && !few_rows(M, N, K));
                    }
            std::printf("%d %d %d %d", wrong, (int)tn_shape(16, 16, 32768, few_rows_alone(16, 16, 32768)).blocks,
                        (int)tn_shape(16, 16, 32768, few_rows(16, 16, 32768)).blocks, (int)tn_shape(16, 16, 1000, few_rows_alone(16, 16, 1000)).blocks);
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "0 256 512 16".split(), (r.returncode, r.stdout, r.stderr)


def test_equal_shares_of_the_columns(tmp_path):
    """Equal shares of the columns only where their pieces meet in a cache; with a mask that is the L2s, unless the product takes longer."""
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include <initializer_list>
        #include "launch_rules.h"
        using namespace gcn;
        int main() {
            std::printf("%d %d %d %d %d %d ", equal_shares(120000, 80, 64, false, 4), equal_shares(120000, 80, 16, true, 4), equal_shares(20000, 80, 16, true, 4),
                        equal_shares(120000, 80, 256, true, 4), equal_shares(326000, 80, 41, true, 4), equal_shares(1000000, 96, 16, false, 4));
            int wrong = 0;
            for (int64_t M : {64, 20000, 65000, 200000, 1000000})
                for (int64_t N = 1; N <= 600; ++N)
                    for (int NT : {1, 2, 3, 4, 8, 16})
                        for (int mask = 0; mask < 2; ++mask) {
                            if (NT > (N + 15) / 16) continue;
                            const int got = equal_shares(M, N, 32, mask, NT);
                            if (got == 0) continue;
                            const int64_t tiles = (N + 15) / 16, shares = (tiles + NT - 1) / NT;
                            wrong += got > NT || got > 4 || (tiles + got - 1) / got != shares;
                        }
            std::printf("%d", wrong);
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "3 0 3 3 0 0 0".split(), (r.returncode, r.stdout, r.stderr)


def test_single_columns_where_all_wavefronts_have_one_strip(tmp_path):
    r = run_cpp(tmp_path, """
        #include <cstdio>
        #include "launch_rules.h"
        using namespace gcn;
        int main() {
            auto of = [](long rows, long k) { return (int)single_columns((rows + 15) / 16, k, 256); };
            std::printf("%d %d %d %d %d %d %d", of(32768, 409), of(32769, 409), of(65536, 300), of(65537, 300), of(40000, 299), of(30000, 700), of(200000, 700));
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == "0 1 1 0 0 0 0".split(), (r.returncode, r.stdout, r.stderr)
