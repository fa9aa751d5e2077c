"""The split of an attention call over workgroups, as host code by itself: the
plan for mixed lengths stays inside its tables and the workspace, and gives
every chunk of every head to exactly one workgroup."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_23843_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <vector>
#include "attention_plan.h"
using namespace pkv;

static int most_slots = 0;

static void check(int B, int Hkv, int P, const std::vector<int32_t> &len, long seed) {
    auto fail = [&](const char *what) {
        std::printf("%s: B=%d Hkv=%d P=%d longest %d (case %ld)\n", what, B, Hkv, P, *std::max_element(len.begin(), len.end()), seed);
        std::exit(1);
    };
    const int64_t longest = std::max<int64_t>(1, ceil_div(*std::max_element(len.begin(), len.end()), P));
    const ChunkPlan full = chunk_plan_equal(B, Hkv, longest);
    auto m = std::make_unique<MixedSeq>();   // on the heap: the sanitizer sees a write past its end
    const ChunkPlan p = chunk_plan(B, Hkv, P, full, len.data(), *m);
    const int64_t nc4 = (full.n_chunks + 3) / 4 * 4;
    if (p.pages_per_chunk < 1 || (int64_t)p.n_chunks * p.pages_per_chunk < longest) fail("pages left out");
    if (p.equal) {
        if (p.n_chunks > nc4) fail("equal plan past the workspace");
        return;
    }
    std::vector<std::vector<int>> seen(B);
    for (int b = 0; b < B; ++b) {
        const int64_t n = std::max<int64_t>(1, ceil_div(len[b], P));
        if (m->len[b] != len[b]) fail("length");
        seen[b].assign(m->first[b + 1] - m->first[b], 0);
        if ((int64_t)seen[b].size() != ceil_div(n, p.pages_per_chunk)) fail("chunks of a sequence");
    }
    const int slots = m->first[B];
    most_slots = std::max(most_slots, slots);
    if (m->first[0] != 0 || slots > kMaxChunkSlots) fail("slots");
    if ((int64_t)slots > B * nc4) fail("past the workspace");
    for (int i = 0; i < slots; ++i) {
        const int b = m->seq_of[i], c = m->chunk_of[i];
        if (b >= B || c >= (int)seen[b].size() || seen[b][c]++) fail("chunk given out twice or not there");
    }
}

int main() {
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    // nearly equal lengths: two chunks each by the plan of equal lengths, 2 B - 1 in all
    for (int B = 2; B <= 255; ++B)
        for (int pages = 2; pages <= 70; ++pages) {
            std::vector<int32_t> len(B, 64 * pages);
            len[pick(0, B - 1)] = pick(0, 64 * (pages - 1));
            check(B, 1, 64, len, pages);
        }
    for (long i = 0; i < 40000; ++i) {
        const int B = pick(0, 2) ? pick(1, 255) : pick(190, 255), Hkv = pick(0, 1) ? 1 : pick(1, 8), P = 16 << pick(0, 2);
        const int top = 1 + (1 << pick(2, 18)), low = pick(0, 3) ? 0 : pick(0, top);
        std::vector<int32_t> len(B);
        for (int32_t &n : len) n = pick(0, 9) ? pick(low, top) : pick(0, top);
        check(B, Hkv, P, len, i);
    }
    std::printf("ok, at most %d slots\n", most_slots);
    return most_slots > 384 ? 0 : 2;   // the plans with two chunks per sequence were reached
}
"""


def test_chunk_plan_stays_inside_its_tables(tmp_path):
    src = tmp_path / "plan.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, str(src), "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], env=env, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
