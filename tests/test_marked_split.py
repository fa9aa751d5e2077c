"""Which wavefront takes which page of the launch over marked pages, as host code
by itself: every page once, and pages that are marked together on many
wavefronts."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_23843_amd", "csrc")

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "marked_split.h"
using namespace pkv;

int main() {
    for (uint32_t waves : {1u, 2u, 3u, 4u, 8u, 60u, 512u, 2047u, 2048u, 3072u})
        for (int64_t n : {1l, 2l, 7l, 64l, 509l, 3072l, 4080l, 8192l, 130496l, 1000003l}) {
            std::vector<int> owner(n, -1);
            for (uint32_t w = 0; w < waves; ++w)
                for (int64_t t = 0; t * waves < n; ++t) {
                    const int64_t i = marked_candidate((uint32_t)t, w, waves, n);
                    if (i == n) continue;
                    if (i < 0 || i > n || owner[i] >= 0) return std::printf("n=%ld waves=%u: candidate %ld\n", (long)n, waves, (long)i), 1;
                    owner[i] = (int)w;
                }
            if (std::count(owner.begin(), owner.end(), -1)) return std::printf("n=%ld waves=%u: left out\n", (long)n, waves), 1;
            // a run of marked candidates in one head, and the same run in each of 32 heads
            for (int64_t heads : {1l, 32l}) {
                const int64_t head = n / heads, run = std::min<int64_t>(head, 256);
                if (run < 8) continue;
                std::vector<int> load(waves, 0);
                for (int64_t h = 0; h < heads; ++h)
                    for (int64_t i = 0; i < run; ++i) ++load[owner[h * head + head / 3 + std::min(i, head - head / 3 - 1)]];
                const int64_t even = (heads * run + waves - 1) / waves;
                const int most = *std::max_element(load.begin(), load.end());
                if (head - head / 3 >= run && most > 4 * even + 3)
                    return std::printf("n=%ld waves=%u heads=%ld: %d on one wavefront, %ld if even\n", (long)n, waves, (long)heads, most, (long)even), 1;
            }
        }
    // the extreme order of heads: their length in candidates a multiple of the wavefronts
    for (int64_t mult : {1l, 2l, 3l}) {
        const uint32_t waves = 3072;
        const int64_t head = mult * waves;
        std::vector<int> load(waves, 0);
        for (uint32_t w = 0; w < waves; ++w)
            for (int64_t t = 0; t < 32 * mult; ++t) {
                const int64_t i = marked_candidate((uint32_t)t, w, waves, 32 * head);
                load[w] += i % head < 256;
            }
        const int most = *std::max_element(load.begin(), load.end());
        if (most > 8) return std::printf("heads of %ld rounds: %d on one wavefront\n", (long)mult, most), 1;
    }
    return 0;
}
"""


def test_marked_pages_are_spread(tmp_path):
    src = tmp_path / "split.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "split")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
