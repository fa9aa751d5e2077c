// How an attention call is cut into chunks of pages: host code without a HIP
// header, so that it also compiles by itself (with a sanitizer, in the tests).
#pragma once

#include <algorithm>
#include <cstdint>

namespace pkv {

constexpr int kMaxBatchArgs = 256;   // sequences whose lengths travel in kernel arguments (batch at most 255)
constexpr int64_t kAttnGroups = 256;   // workgroups aimed at, one per CU

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Sequence lengths of an attention launch and its chunks: each KV head of
// sequence b is split over a number of workgroups, and their partial states
// follow those of the heads before it. With the same number for every head
// (EqualSeq) the grid is (chunk, head); otherwise (MixedSeq) the heads of
// sequence b have first[b + 1] - first[b] chunks and workgroup i * Hkv + h
// serves chunk chunk_of[i] of head h of sequence seq_of[i], longest sequences
// first. Two types and not a flag: the lookups cost a 16 us call 0.2 us also
// where it did not make them.
//
// kMaxChunkSlots: chunks of one KV head over all sequences. chunk_plan stops at
// 256 workgroups or at 1.5 per head, unless equal lengths would give more: with
// N = B * Hkv heads equal lengths give a head ceil(n / ceil(n N / 256)) <=
// ceil(256 / N) chunks, so B of them at most B ceil(256 / B) = 2 B, at B =
// 129..255 and Hkv = 1.
constexpr int kMaxChunkSlots = 2 * kMaxBatchArgs;
struct EqualSeq {
    int32_t len[kMaxBatchArgs];
    int32_t n_chunks;   // read together with the kernel's next argument
};
struct MixedSeq {
    int32_t len[kMaxBatchArgs];
    int32_t first[kMaxBatchArgs + 1];
    uint8_t seq_of[kMaxChunkSlots], chunk_of[kMaxChunkSlots];
};

struct ChunkPlan {
    int pages_per_chunk;
    int n_chunks;   // of the longest sequence
    bool equal;     // every head has n_chunks of them
};

// The plan when every sequence has n_pages pages.
inline ChunkPlan chunk_plan_equal(int B, int Hkv, int64_t n_pages) {
    const int64_t ppc = std::max<int64_t>(1, ceil_div(n_pages * B * Hkv, kAttnGroups));
    return {(int)ppc, (int)ceil_div(n_pages, ppc), true};
}

// The most chunks of a head among plans of equal lengths up to n_pages pages.
// The number is not monotone: 8 heads have 32 chunks of one page at 32 pages and
// 17 of two at 33.
inline int most_chunks(int B, int Hkv, int64_t n_pages) {
    return (int)std::min(n_pages, ceil_div(kAttnGroups, (int64_t)B * Hkv));
}

// The plan for these lengths; `full` is that of equal lengths, all the longest.
// The pages per chunk come from the pages there are, not from the longest
// sequence times the batch: in a batch of mixed lengths the long heads would
// otherwise get as few workgroups as the short ones and finish alone (128 heads
// of 16 sequences of 500 to 16,363 tokens: 91 us with two chunks each, 66 us
// with one to five; 32 sequences of one KV head and up to 32,001 tokens: 43 ->
// 32 us). A chunk beyond one per CU would start when another ends, so chunks
// grow until their number is at most 256, or half as many again as heads when
// there are more heads than that, and fits the partial states of a workspace
// sized for the longest sequence; they stop at the chunks of equal lengths. And
// a head is not cut into more than 32 chunks that equal lengths would not give
// it, since its merge takes a round trip per 32 (8 sequences of one KV head and
// up to 65,001 tokens: 28.6 us with 32, 29.4 us with 79). The grid holds the
// chunks there are: with workgroups that find nothing to do in it the same plan
// lost (91 -> 96 us). `out` is written only where the plan is not `equal`.
inline ChunkPlan chunk_plan(int B, int Hkv, int P, const ChunkPlan &full, const int32_t *len, MixedSeq &out) {
    if (std::all_of(len, len + B, [&](int32_t n) { return n == len[0]; })) return full;
    const int64_t heads = (int64_t)B * Hkv;
    const int64_t most = std::min({std::max(kAttnGroups, heads + heads / 2), heads * ((full.n_chunks + 3) / 4 * 4),
                                   (int64_t)kMaxChunkSlots * Hkv});
    auto pages = [&](int b) { return std::max<int64_t>(1, ceil_div(len[b], P)); };
    int64_t total = 0, longest = 1;
    for (int b = 0; b < B; ++b) {
        total += pages(b);
        longest = std::max(longest, pages(b));
    }
    int64_t ppc = std::max(ceil_div(total * Hkv, kAttnGroups), ceil_div(longest, std::max(32, full.n_chunks)));
    for (;; ppc += std::max<int64_t>(1, ppc / 32)) {
        int64_t n = 0;
        for (int b = 0; b < B; ++b) n += ceil_div(pages(b), ppc);
        if (n * Hkv <= most || ppc >= full.pages_per_chunk) break;
    }
    ChunkPlan p;
    p.pages_per_chunk = (int)std::min<int64_t>(ppc, full.pages_per_chunk);
    p.n_chunks = (int)ceil_div(longest, p.pages_per_chunk);
    p.equal = true;   // of different lengths, but the same number of chunks
    int64_t slots = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = ceil_div(pages(b), p.pages_per_chunk);
        slots += n;
        if (n != p.n_chunks) p.equal = false;
    }
    if (p.equal) return p;
    // out of reach by the bound above; the plan of equal lengths needs no table
    if (slots > kMaxChunkSlots || p.n_chunks > 256) return full;
    int order[kMaxBatchArgs];
    out.first[0] = 0;
    for (int b = 0; b < B; ++b) {
        out.len[b] = len[b];
        out.first[b + 1] = out.first[b] + (int)ceil_div(pages(b), p.pages_per_chunk);
        order[b] = b;
    }
    std::sort(order, order + B, [&](int x, int y) { return len[x] != len[y] ? len[x] > len[y] : x < y; });
    int i = 0;
    for (int x = 0; x < B; ++x)
        for (int c = 0; c < out.first[order[x] + 1] - out.first[order[x]]; ++c, ++i) {
            out.seq_of[i] = (uint8_t)order[x];
            out.chunk_of[i] = (uint8_t)c;
        }
    return p;
}

}  // namespace pkv
