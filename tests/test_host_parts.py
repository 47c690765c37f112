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
