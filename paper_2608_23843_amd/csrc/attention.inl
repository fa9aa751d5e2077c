// Mixed-page decode attention (Eq. (4) for factor pages, the same state from
// K and V for dense pages, Eq. (5) to merge) -- split phase and combine.
//
// Work is split flash-decoding style: each workgroup owns one (sequence, KV
// head) and a contiguous chunk of pages, keeps the running (m, l, O) state
// of the g query heads of that KV head, and writes it as a partial; the last
// workgroup of a head merges its partials with the Eq. (5) rescaling.
// Scores are kept in the base-2 domain (s * log2(e) / sqrt(d)) so every
// exponential is one exp2.
// Included by pkv_kernels.hip.

namespace pkv {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Workspace of one call. It starts with the per-head words that must be zero
// when a call begins and that every call returns to zero: one merge counter
// per (sequence, KV head) `head`, then one page-claim word per head on its
// own 256-byte line. Their offsets depend only on the number of heads, so a
// workspace sized for the longest sequence can be shared by calls of any
// length. The partial states follow, for each head, chunk c and query qi of
// the group: O[head][c][qi][k], the max M[head][c][qi] (log2 units) and the
// normalizer L[head][c][qi], the chunks of head after head (HeadChunks says
// which are a head's), so that each workgroup's partial is one
// contiguous block (whole cache lines written, no line shared between
// workgroups) and the merge reads one chunk per load across consecutive
// lanes. The partials are fully written by every call before they are read.
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Partials {
    float *o, *m, *l;
    unsigned int *counters;  // chunks published, per head
    unsigned int *claims;    // pages handed out, per head (streaming kernel), one per 256 bytes
    __host__ __device__ unsigned int *claim(int64_t head) const { return claims + head * 64; }
    int nc, nc4, g, d;
    __device__ int64_t oi(int64_t c, int qi, int k) const { return (c * g + qi) * d + k; }
    __device__ int64_t mi(int64_t c, int qi) const { return c * g + qi; }
};

// A head's chunks: `n` partial states from index `first` on.
struct HeadChunks {
    int64_t first;
    int n;
};

__host__ __device__ inline int64_t round256(int64_t b) { return (b + 255) / 256 * 256; }

// Bytes of the zero-on-entry words for `heads` heads.
__host__ __device__ inline int64_t counter_bytes(int64_t heads) { return round256(heads * 4) + heads * 256; }
// Bytes of the partial states.
__host__ __device__ inline int64_t partial_state_bytes(int64_t heads, int n_chunks, int g, int d) {
    const int64_t nc4 = (n_chunks + 3) / 4 * 4;
    return round256(heads * g * d * nc4 * 4) + 2 * round256(heads * g * nc4 * 4);
}
__host__ __device__ inline int64_t partials_bytes(int64_t heads, int n_chunks, int g, int d) {
    return counter_bytes(heads) + partial_state_bytes(heads, n_chunks, g, d);
}

// counters: a region of counter_bytes(heads_cap) bytes (heads_cap >= heads)
// laid out as the counters of heads_cap heads; states: the partial states.
__host__ __device__ inline Partials make_partials(void *counters, int64_t heads_cap, void *states, int64_t heads,
                                                  int n_chunks, int g, int d) {
    Partials p;
    p.nc = n_chunks;
    p.nc4 = (n_chunks + 3) / 4 * 4;
    p.g = g;
    p.d = d;
    p.counters = (unsigned int *)counters;
    p.claims = (unsigned int *)((char *)counters + round256(heads_cap * 4));
    char *c = (char *)states;
    p.o = (float *)c;
    c += round256(heads * g * d * p.nc4 * 4);
    p.m = (float *)c;
    c += round256(heads * g * p.nc4 * 4);
    p.l = (float *)c;
    return p;
}
// A caller's workspace: the counters of `heads` heads, then the states.
__host__ __device__ inline Partials make_partials(void *ws, int64_t heads, int n_chunks, int g, int d) {
    return make_partials(ws, heads, (char *)ws + counter_bytes(heads), heads, n_chunks, g, d);
}

__device__ inline HeadChunks head_chunks(const EqualSeq &, const Partials &pp, const AttnWork &w, int) {
    return {w.head * pp.nc4, pp.nc};
}
__device__ inline HeadChunks head_chunks(const MixedSeq &seq, const Partials &, const AttnWork &w, int Hkv) {
    return {(int64_t)seq.first[w.b] * Hkv + w.h * w.n_chunks, w.n_chunks};
}

// One workgroup per chunk.
inline dim3 attention_grid(const Geo &g, const EqualSeq &seq) { return dim3(seq.n_chunks, g.B * g.Hkv); }
inline dim3 attention_grid(const Geo &g, const MixedSeq &seq) { return dim3(seq.first[g.B] * g.Hkv); }

// ---- combine: Eq. (5) across the chunks of one head, then normalize -----------
//
// Fused into the split kernels: every workgroup publishes its partial, then
// bumps the head's counter; the workgroup that brings it to n_chunks merges
// the head and resets the counter to zero for the next call. No workgroup
// ever waits on another, so the pattern cannot stall.
//
// Partials and counters are written and read with device-scope atomic
// accesses (relaxed), which the caches keep coherent across the chip's
// L2 slices one access at a time. A device-scope fence would instead write
// back and invalidate a whole L2 per workgroup, stalling every other
// workgroup's stream on that slice. Order comes from waiting for the
// workgroup's own stores to complete before the counter is bumped.
__device__ inline void st_dev(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float ld_dev(const float *p) {
    return __hip_atomic_load(const_cast<float *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by every thread of an NT-thread workgroup after its partial stores.
// The workgroup that completes the head merges all of its chunks (Eq. (5)).
// Chunks are folded in groups of kMergeGroup. A group's maxima and
// normalizers are read once, one or two per thread, and passed through LDS;
// each thread's kMergeGroup partial outputs are in flight with them, so a
// group costs one round trip to memory (kMergeGroup + 2 loads stay within a
// wave's 63 outstanding vector loads). The loads are unconditional (a chunk
// past the end reads the last one and is masked), which keeps this code
// short: it runs once per launch, from a cold instruction cache.
constexpr int kMergeGroup = 32;

// The fold of the last workgroup with 16-byte partial loads, for shapes whose
// F = G d / 4 groups of four outputs divide the workgroup into R lanes each:
// thread (f, r) folds chunks r, r + R, ... of output group f (one coherent
// 16-byte load per chunk, J per group of kMergeGroup chunks, loads past the
// last chunk read it again and are masked), every lane of a query uses the
// same running max (the group's maxima through LDS), and the R partial sums
// of an output group are added through LDS at the end. s_mg, s_lg: the
// group maxima and normalizers (16 x kMergeGroup floats each); red: 5 NT
// floats of LDS for the sums, 16-byte aligned.
template <int NT, int R>
__device__ void merge_vec(const Geo &g, int64_t head, const Partials &pp, HeadChunks hc, float *out, float *lse, int64_t T,
                          float *s_mg, float *s_lg, float *red) {
    constexpr int J = (kMergeGroup + R - 1) / R;
    constexpr int MLT = (16 * kMergeGroup + NT - 1) / NT;
    f32x4 *s_ra = (f32x4 *)red;
    float *s_rl = red + 4 * NT;
    const int tid = threadIdx.x;
    const int nc = hc.n, G = g.g, d = g.d;
    const int F = NT / R;
    const int f = tid % F, r = tid / F;
    const int q = (4 * f) / d, k = (4 * f) % d;
    const uint32_t cs = (uint32_t)(G * d) * 4u;   // chunk stride in bytes
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        pp.o + pp.oi(hc.first, 0, 0), (short)0, (int)((uint32_t)hc.n * cs), 0x00020000);
    float M = -INFINITY, L = 0.f;
    f32x4 A = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nc; c0 += kMergeGroup) {
        float mreg[MLT], lreg[MLT];
#pragma unroll
        for (int i = 0; i < MLT; ++i) {
            const int t = tid + i * NT;
            const int qm = min(t / kMergeGroup, G - 1), cu = min(c0 + t % kMergeGroup, nc - 1);
            mreg[i] = ld_dev(pp.m + pp.mi(hc.first + cu, qm));
            lreg[i] = ld_dev(pp.l + pp.mi(hc.first + cu, qm));
        }
        f32x4 ov[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t c = (uint32_t)min(c0 + r + R * j, nc - 1);
            ov[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ro, c * cs + 16u * (uint32_t)f, 0, 16));
        }
        __syncthreads();   // the previous group's maxima have been read
#pragma unroll
        for (int i = 0; i < MLT; ++i) {
            const int t = tid + i * NT;
            if (t < 16 * kMergeGroup) {
                s_mg[t] = (t % kMergeGroup) < nc - c0 ? mreg[i] : -INFINITY;
                s_lg[t] = lreg[i];
            }
        }
        __syncthreads();
        const float *mg = s_mg + q * kMergeGroup, *lg = s_lg + q * kMergeGroup;
        float Mg = M;
        for (int u = 0; u < kMergeGroup; u += 4) {
            const f32x4 m4 = *(const f32x4 *)(mg + u);
            Mg = fmaxf(Mg, fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
        }
        if (Mg == -INFINITY) continue;   // no tokens in any chunk so far
        const float sc = __builtin_amdgcn_exp2f(M - Mg);
        L *= sc;
        A *= sc;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int u = r + R * j;   // chunk c0 + u; at or past nc its maximum is -inf
            const float wgt = u < kMergeGroup ? __builtin_amdgcn_exp2f(mg[u] - Mg) : 0.f;
            if (u < kMergeGroup) L = fmaf(wgt, lg[u], L);
            A += wgt * ov[j];
        }
        M = Mg;
    }
    s_ra[tid] = A;
    s_rl[tid] = L;
    __syncthreads();
    if (r == 0) {
#pragma unroll
        for (int i = 1; i < R; ++i) {
            A += s_ra[i * F + f];
            L += s_rl[i * F + f];
        }
        const bool empty = T <= 0 || !(L > 0.f);
        const int b = (int)(head / g.Hkv), h = (int)(head % g.Hkv);
        float *o = out + ((int64_t)b * g.Hq + h * G + q) * d + k;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = empty ? 0.f : A[i] / L;
        if (lse && k == 0) lse[(int64_t)b * g.Hq + h * G + q] = empty ? -INFINITY : (M + log2f(L)) * kLn2;
    }
}

// red: at least 5 NT floats of LDS the caller no longer needs (16-byte
// aligned), or null: the fold with 16-byte loads needs them.
template <int NT>
__device__ void publish_and_merge(const Geo &g, int64_t head, const Partials &pp, HeadChunks hc, float *out, float *lse,
                                  int64_t T, float *red = nullptr) {
    constexpr int kMaxG = 16;                                      // the kernels' query-group limit
    constexpr int MLT = (kMaxG * kMergeGroup + NT - 1) / NT;       // group maxima per thread
    __shared__ unsigned int s_prev;
    __shared__ float s_mg[kMaxG * kMergeGroup], s_lg[kMaxG * kMergeGroup];
    const int tid = threadIdx.x;
    const int nc = hc.n;
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this thread's partial stores have completed
    __syncthreads();
    if (tid == 0) s_prev = __hip_atomic_fetch_add(&pp.counters[head], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_prev != (unsigned int)(nc - 1)) return;

    const int G = g.g, d = g.d;
    bool done = false;
    // only where the per-output fold below would take several passes (G d >
    // NT, so two or three lanes per output group): at batch 1 (G d = NT, 32
    // chunks) that fold measured faster
    if (red && G * d > NT && (G * d) % 4 == 0 && NT % (G * d / 4) == 0) {
        switch (NT / (G * d / 4)) {
        case 2: merge_vec<NT, 2>(g, head, pp, hc, out, lse, T, s_mg, s_lg, red); done = true; break;
        case 3: merge_vec<NT, 3>(g, head, pp, hc, out, lse, T, s_mg, s_lg, red); done = true; break;
        default: break;
        }
    }
    if (done) {
        if (tid == 0) {
            __hip_atomic_store(&pp.counters[head], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(pp.claim(head), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    const int b = (int)(head / g.Hkv), h = (int)(head % g.Hkv);
    // the same trip counts in every thread: the group loop holds barriers
    for (int base = 0; base < G * d; base += NT) {
        const int idx = min(base + tid, G * d - 1);   // threads past the end redo the last output, unstored
        const int qi = idx / d, k = idx % d;
        const float *op = pp.o + pp.oi(hc.first, qi, k);
        const int co = G * d;   // chunk stride of the outputs
        float M = -INFINITY, L = 0.f, A = 0.f;
        for (int c0 = 0; c0 < nc; c0 += kMergeGroup) {
            float mreg[MLT], lreg[MLT];
#pragma unroll
            for (int i = 0; i < MLT; ++i) {
                const int t = tid + i * NT;
                const int qm = min(t / kMergeGroup, G - 1), cu = min(c0 + t % kMergeGroup, nc - 1);
                mreg[i] = ld_dev(pp.m + pp.mi(hc.first + cu, qm));
                lreg[i] = ld_dev(pp.l + pp.mi(hc.first + cu, qm));
            }
            float ov[kMergeGroup];
#pragma unroll
            for (int u = 0; u < kMergeGroup; ++u) ov[u] = ld_dev(op + (uint32_t)(min(c0 + u, nc - 1) * co));
            __syncthreads();   // the previous group's maxima have been read
#pragma unroll
            for (int i = 0; i < MLT; ++i) {
                const int t = tid + i * NT;
                if (t < kMaxG * kMergeGroup) {
                    s_mg[t] = (t % kMergeGroup) < nc - c0 ? mreg[i] : -INFINITY;
                    s_lg[t] = lreg[i];
                }
            }
            __syncthreads();
            const float *mg = s_mg + qi * kMergeGroup, *lg = s_lg + qi * kMergeGroup;
            float Mg = M;
#pragma unroll
            for (int u = 0; u < kMergeGroup; ++u) Mg = fmaxf(Mg, mg[u]);
            if (Mg == -INFINITY) continue;   // no tokens in any chunk so far
            // arguments <= 0 with Mg finite: the hardware exp2 gives 0 for -inf
            // (an empty chunk, or no state yet) and needs no range fix-up
            const float sc = __builtin_amdgcn_exp2f(M - Mg);
            L *= sc;
            A *= sc;
#pragma unroll
            for (int u = 0; u < kMergeGroup; ++u) {
                const float wgt = __builtin_amdgcn_exp2f(mg[u] - Mg);
                L = fmaf(wgt, lg[u], L);
                A = fmaf(wgt, ov[u], A);
            }
            M = Mg;
        }
        if (base + tid < G * d) {
            const bool empty = T <= 0 || !(L > 0.f);
            out[((int64_t)b * g.Hq + h * G + qi) * d + k] = empty ? 0.f : A / L;
            if (lse && k == 0) lse[(int64_t)b * g.Hq + h * G + qi] = empty ? -INFINITY : (M + log2f(L)) * kLn2;
        }
    }
    if (tid == 0) {
        __hip_atomic_store(&pp.counters[head], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(pp.claim(head), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---- any supported geometry, fp32 or bf16 storage ------------------------------
//
// Pages in fp32 arithmetic from the stored values, one page per wavefront at a
// time: all products are 16x16x4 fp32 matrix products with the query group in
// N. Lane (n, q) = (lane % 16, lane / 16) holds rows 4 q + i of column n of a
// 16-row tile in register i, which is the right operand of the next product's
// i-th step (ranks, tokens or dims 4 q + i), so the chain
//   Z^T = R_K Q^T, S^T = L_K Z^T, Y^T = L_V^T E^T, O^T += R_V^T Y^T
// (S^T = K Q^T, O^T += V^T E^T on dense pages) moves no data between lanes and
// every left operand is four consecutive entries of a stored row. Rows, ranks
// and tokens past the end are read as zero.
// Eight wavefronts per workgroup, about 256 workgroups: each wavefront's loads
// of a phase are in flight together and it waits on memory four times a page,
// so what bounds a short cache is the launch, those waits and the merge, a
// long one its loads. The tile loops over ranks stay loops, with Z and Y passed
// through LDS: the code runs from a cold instruction cache, and unrolled over
// four rank tiles it took longer than the loads. A workgroup of 256 threads
// sharing one page through LDS, with one entry per load, a barrier per phase and
// 1,024 workgroups, took 66 us on a 4K fp32 cache of 8 KV heads (21 MB) against
// 16; at 32K 342 against 41, at 128K 956 against 165 (605 MB), with d = 256 and
// rank 48 at 32K 707 against 129 (504 MB), d = 192 at 4K 69 against 34, and on
// bf16 pages of rank 64 at 128K 2,047 against 276 (805 MB). With 512 or 1,024
// workgroups this kernel loses at all of these (4K 25 and 36 us, 128K 175 and
// 202, d = 256 150 and 211): the merge grows and a head's waves share less.
// 16-token pages of 64 dims alone gain from 512 (32K: 45 -> 38 us).

constexpr int kGenWaves = 8, kGenThreads = 64 * kGenWaves;

// Four consecutive stored entries as fp32.
__device__ __forceinline__ f32x4 gen_ld4(const float *p) { return *(const f32x4 *)p; }
__device__ __forceinline__ f32x4 gen_ld4(const uint16_t *p) {
    const uint2 w = *(const uint2 *)p;
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
}
// c += a b over the 16 entries of four steps.
__device__ __forceinline__ f32x4 gen_mfma(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
    return c;
}
// Maximum and sum over the four lane rows.
__device__ __forceinline__ float gen_qmax(float v) {
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float gen_qsum(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// LDS floats: the query group (16 rows, padded) and each wavefront's Z or Y (16
// queries x 64 ranks, padded); then, in their place, the states of four
// wavefronts.
constexpr int kGenLdZ = 68;
inline int gen_lds(const Geo &g, int dims) {
    return std::max(16 * (dims + 4) + kGenWaves * 16 * kGenLdZ, 4 * g.g * g.d);
}

// Order of a wavefront's LDS accesses (they execute in order; this keeps the
// compiler from moving them across).
__device__ __forceinline__ void gen_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// 16 stored rows times the query group over d dims: lane (n, q) reads row n at
// p. Past d (d <= 16 DT) the last dims are read again and not used.
template <int DT, typename T>
__device__ __forceinline__ f32x4 gen_rows(const T *p, const float *sq, int d) {
    f32x4 a[DT], c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DT; ++s) a[s] = gen_ld4(p + min(16 * s, d - 16));
#pragma unroll
    for (int s = 0; s < DT; s += 2)   // d is a multiple of 32, above 8 DT (32 for DT = 4)
        if (s < (DT == 4 ? 2 : DT / 2 + 2) || 16 * s < d) {
            c = gen_mfma(a[s], *(const f32x4 *)(sq + 16 * s), c);
            c = gen_mfma(a[s + 1], *(const f32x4 *)(sq + 16 * s + 16), c);
        }
    return c;
}
// o[t] += 16 stored columns times b: lane (n, q) reads entries of dim 16 t + n
// at p + t * step, of which the first `live` count. Tiles past d repeat the
// first and are not used.
template <int DT, typename T>
__device__ __forceinline__ void gen_cols(const T *p, int step, int d, int live, f32x4 b, f32x4 (&o)[DT]) {
    f32x4 a[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) a[t] = gen_ld4(p + (16 * t < d ? t * step : 0));
#pragma unroll
    for (int t = 0; t < DT; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a[t][i] = i < live ? a[t][i] : 0.f;
        o[t] = gen_mfma(a[t], b, o[t]);
    }
}

// DT: 16-dim tiles of the output held per wavefront (d <= 16 DT).
template <typename TD, typename TF, int DT, typename Seq>
__global__ __launch_bounds__(kGenThreads) void k_attn_generic(Geo g, const pkv_page *table, const char *dense,
                                                              const char *factor, const TD *q, Seq seq, int ppc,
                                                              Partials pp, float *out, float *lse) {
    extern __shared__ __align__(16) float gen_smem[];
    __shared__ float sM[kGenWaves][16], sL[kGenWaves][16];
    const AttnWork work = attn_work(seq, g.Hkv);
    const HeadChunks hc = head_chunks(seq, pp, work, g.Hkv);
    const int chunk = work.chunk, n_chunks = work.n_chunks, b = work.b, h = work.h;
    const int64_t head = work.head;
    const int G = g.g, d = g.d, P = g.P, PT = P / 16;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, r4q = 4 * (lane >> 4);
    const int64_t T = seq.len[b];
    const int n_pages = (int)ceil_div(T, P);
    const int j0 = chunk * ppc, j1 = min(j0 + ppc, n_pages);
    const float c2 = kLog2e / sqrtf((float)d);
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};

    constexpr int ldq = 16 * DT + 4;
    for (int i = tid; i < 16 * 16 * DT; i += kGenThreads) {
        const int qi = i / (16 * DT), k = i % (16 * DT);
        gen_smem[qi * ldq + k] = qi < G && k < d ? to_f32(q[((int64_t)b * g.Hq + (int64_t)h * G + qi) * d + k]) : 0.f;
    }
    __syncthreads();
    const float *sq = gen_smem + n * ldq + r4q;
    float *sz = gen_smem + 16 * ldq + (wave * 16 + n) * kGenLdZ + r4q;

    float m = -INFINITY, l = 0.f;   // of query n
    f32x4 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = zero4;
    for (int j = j0 + wave; j < j1; j += kGenWaves) {
        const pkv_page e = table[head * g.max_pages + j];
        const int kind = __builtin_amdgcn_readfirstlane((int)e.kind);
        const int64_t slot = __builtin_amdgcn_readfirstlane(e.slot);
        const int rows = min(P, (int)(T - (int64_t)j * P));
        const int rk = __builtin_amdgcn_readfirstlane((int)e.rank_k), rv = __builtin_amdgcn_readfirstlane((int)e.rank_v);
        const int rk4 = r4(rk), rv4 = r4(rv);
        const FactorLayout fl = factor_layout(P, d, rk, rv);
        const TF *Ak = (const TF *)(factor + slot * g.factor_slot_bytes);
        const TD *K = (const TD *)(dense + slot * g.dense_slot_bytes);
        f32x4 st[4];   // scores, then weights: tokens 16 t + 4 q + i
#pragma unroll
        for (int t = 0; t < 4; ++t) st[t] = zero4;
        if (kind == PKV_FACTOR) {
#pragma unroll 1
            for (int t = 0; t < rk; t += 16) {
                const bool in = t + n < rk;   // rows past the rank are read as row 0 and dropped
                const f32x4 z = gen_rows<DT>(Ak + fl.bk + (in ? (t + n) * d : 0) + r4q, sq, d);
                *(f32x4 *)(sz + t) = f32x4{t + r4q < rk ? z[0] : 0.f, t + r4q + 1 < rk ? z[1] : 0.f,
                                           t + r4q + 2 < rk ? z[2] : 0.f, t + r4q + 3 < rk ? z[3] : 0.f};
            }
            gen_lds_order();
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < PT)
#pragma unroll 1
                    for (int s = 0; s < rk; s += 16) {
                        const bool in = s + r4q < rk4;
                        f32x4 a = gen_ld4(Ak + (16 * t + n) * rk4 + (in ? s + r4q : 0));
                        st[t] = gen_mfma(in ? a : zero4, *(const f32x4 *)(sz + s), st[t]);
                    }
        } else if (kind == PKV_DENSE) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < PT) st[t] = gen_rows<DT>(K + (16 * t + n) * d + r4q, sq, d);
        } else {
            if (lane == 0) raise_status(PKV_DEV_BAD_PAGE);
            continue;
        }
        // online softmax over the page's tokens
        float pm = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                st[t][i] = 16 * t + r4q + i < rows ? st[t][i] * c2 : -INFINITY;
                pm = fmaxf(pm, st[t][i]);
            }
        const float m_new = fmaxf(m, gen_qmax(pm));
        const float alpha = m == -INFINITY ? 0.f : exp2f(m - m_new);
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                st[t][i] = st[t][i] == -INFINITY ? 0.f : exp2f(st[t][i] - m_new);
                sum += st[t][i];
            }
        l = fmaf(l, alpha, gen_qsum(sum));
        m = m_new;
        if (__any(alpha != 1.f))
#pragma unroll
            for (int t = 0; t < DT; ++t) o[t] *= alpha;
        if (kind == PKV_FACTOR) {
#pragma unroll 1
            for (int t = 0; t < rv; t += 16) {
                const bool in = t + n < rv;
                const TF *Ar = Ak + fl.avt + (in ? (t + n) * P : 0) + r4q;
                f32x4 a[4], y = zero4;
#pragma unroll
                for (int s = 0; s < 4; ++s) a[s] = gen_ld4(Ar + 16 * min(s, PT - 1));
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (s < PT) y = gen_mfma(a[s], st[s], y);
                *(f32x4 *)(sz + t) = f32x4{t + r4q < rv ? y[0] : 0.f, t + r4q + 1 < rv ? y[1] : 0.f,
                                           t + r4q + 2 < rv ? y[2] : 0.f, t + r4q + 3 < rv ? y[3] : 0.f};
            }
            gen_lds_order();
#pragma unroll 1
            for (int s = 0; s < rv; s += 16) {
                const bool in = s + r4q < rv4;
                gen_cols<DT>(Ak + fl.bvt + n * rv4 + (in ? s + r4q : 0), 16 * rv4, d, in ? 4 : 0, *(const f32x4 *)(sz + s), o);
            }
        } else {
            const TD *Vt = K + (int64_t)P * d + n * P + r4q;
#pragma unroll
            for (int s = 0; s < 4; ++s)   // tokens not yet written are dropped
                if (s < PT) gen_cols<DT>(Vt + 16 * s, 16 * P, d, rows - (16 * s + r4q), st[s], o);
        }
        gen_lds_order();
    }

    // the eight wave states merged (Eq. (5)): wavefronts 4..7 hand theirs to 0..3
    if (r4q == 0) {
        sM[wave][n] = m;
        sL[wave][n] = l;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kGenWaves; ++w) M = fmaxf(M, sM[w][n]);
    const float f = m == -INFINITY ? 0.f : exp2f(m - M);
    float *mine = gen_smem + (int64_t)((wave & 3) * G + n) * d + r4q;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        if (n < G && (pass == 0) == (wave >= 4)) {
#pragma unroll
            for (int t = 0; t < DT; ++t)
                if (16 * t < d) {
                    f32x4 *s = (f32x4 *)(mine + 16 * t);
                    *s = pass == 0 ? o[t] * f : o[t] * f + *s;
                }
        }
        __syncthreads();
    }
    const int b0 = b * g.Hq + h * G;
    for (int i = 4 * tid; i < G * d; i += 4 * kGenThreads) {
        const int qi = i / d, k = i - qi * d;
        f32x4 v = *(const f32x4 *)(gen_smem + i);
#pragma unroll
        for (int w = 1; w < 4; ++w) v += *(const f32x4 *)(gen_smem + w * G * d + i);
        float Mq = -INFINITY, Lq = 0.f;
#pragma unroll
        for (int w = 0; w < kGenWaves; ++w) Mq = fmaxf(Mq, sM[w][qi]);
#pragma unroll
        for (int w = 0; w < kGenWaves; ++w) Lq += sM[w][qi] == -INFINITY ? 0.f : sL[w][qi] * exp2f(sM[w][qi] - Mq);
        if (n_chunks == 1) {   // the head's only workgroup
            const bool empty = T <= 0 || !(Lq > 0.f);
#pragma unroll
            for (int u = 0; u < 4; ++u) out[(int64_t)(b0 + qi) * d + k + u] = empty ? 0.f : v[u] / Lq;
            if (lse && k == 0) lse[b0 + qi] = empty ? -INFINITY : (Mq + log2f(Lq)) * kLn2;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) st_dev(&pp.o[pp.oi(hc.first + chunk, qi, k + u)], v[u]);
            if (k == 0) {
                st_dev(&pp.m[pp.mi(hc.first + chunk, qi)], Mq);
                st_dev(&pp.l[pp.mi(hc.first + chunk, qi)], Lq);
            }
        }
    }
    if (n_chunks == 1) return;
    __syncthreads();
    publish_and_merge<kGenThreads>(g, head, pp, hc, out, lse, T, gen_smem);   // at least 9,792 floats of LDS
}

}  // namespace pkv
