"""Host-side parts of the library that need no GPU, compiled by themselves with the host compiler."""
import os
import subprocess
import textwrap

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_03300_amd", "csrc")


def run_cpp(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(textwrap.dedent(body))
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
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
                const int b = c.best_blocks(rows, l, t.n, 1, &split);
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
                    c.best_blocks(l, c.lines(l), n, 1, &x);
                    if (!std::isfinite(x) || !std::isfinite(c.sweep(l, c.lines(l), n, n, 8, 511, 5, 3, &hb)) || hb < 1) std::printf("bad ");
                }
            c.best_blocks(none, c.lines(none), 1, 1, &x);
            std::printf(std::isfinite(x) ? "ok" : "bad");
        }
    """)
    assert r.returncode == 0 and r.stdout.split() == ["111"] * 8 + ["ok"], (r.returncode, r.stdout, r.stderr)


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
                const int b = c.best_blocks(rows, c.lines(rows), t.n, t.usual, &cost);
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
                        while (parts < 20 && !c.as_exact(l, 1, 1, parts, 8, normalised)) ++parts;
                        if (SpmmCost::sweep_error(mean, parts) > SpmmCost::split_error(mean, f <= 16 ? 32 : 64, 1) || parts < 2 || parts > 8)
                            std::printf("mean %d f %d: %d sums ", mean, f, parts);
                    }
                    if (!c.as_exact(l, 4, 4, 0, 8, true) || c.as_exact(l, 4, 2, 0, 8, true)) std::printf("blocks %d %d ", mean, f);
                }
            std::printf("done");
        }
    """)
    assert r.returncode == 0 and r.stdout == "done", (r.returncode, r.stdout, r.stderr)
