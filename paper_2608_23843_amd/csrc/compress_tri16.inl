// The direct decomposition of compress_tri.inl for bf16 pages of 16 tokens:
// one wavefront takes the K and V halves of two pages. A half's 16x16 Gram
// matrix is one block of the four-block 16x16x1 fp32 product, four registers a
// lane: lane (n, q) = (lane % 16, lane / 16) holds rows 4 q + i of column n of
// half b in register 4 b + i. Vectors are one element per lane (lane 16 b + c:
// element c of half b), which is also the operand form of that product, so the
// rank-2 update of all four halves is two products with no data movement, and
// the products G u of the four halves are 16 fmas and three swaps (fp32 factors:
// in fp64 on the vector ALU). Pages whose eigenvalues cannot be told apart are marked for
// k_compress.
// What bounds it: vector-ALU issue and, with one page's work so short, the
// page reads of the first and last phase. Measured against Jacobi in fp32
// vector code (k_compress): a 16K prompt of 8 KV heads at (r_K, r_V) = (9, 9)
// 510 -> 69 us.
// Included by pkv_kernels.hip after compress_tri.inl.

namespace pkv {

typedef __bf16 c16_bf16x4 __attribute__((ext_vector_type(4)));
typedef short c16_s16x4 __attribute__((ext_vector_type(4)));
typedef float c16_f32x4 __attribute__((ext_vector_type(4)));

constexpr int kC16ZStride = 20;   // LDS row of a token's 16 vector entries
// LDS floats: 14 reflectors of 16 elements per half, (d, e) and (d, e^2) pairs
// of T (f64: and a step's u and w in fp64); then, in the same place, the vectors
// by token row.
constexpr int c16_lds(bool f64) {
    const int tri = 4 * 14 * 16 + 2 * 128 + (f64 ? 256 : 0), z = 4 * 16 * kC16ZStride;
    return tri > z ? tri : z;
}

__device__ __forceinline__ cq_f32x16 c16_outer(float a, float b, cq_f32x16 c) {
    return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ c16_f32x4 c16_mfma4(float a, float b, c16_f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Odd 16-lane rows of x exchanged with even rows of y.
__device__ __forceinline__ ct_pair c16_swap16(float x, float y) {
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return {__uint_as_float(t[0]), __uint_as_float(t[1])};
}
// Lane row b gets the sum over the four lane rows of t[b].
__device__ __forceinline__ float c16_row_sums(float t0, float t1, float t2, float t3) {
    const ct_pair x = ct_swap32(t0, t2), y = ct_swap32(t1, t3);
    const ct_pair s = c16_swap16(x.a + x.b, y.a + y.b);
    return s.a + s.b;
}

__device__ __forceinline__ double c16_row_sums(double t0, double t1, double t2, double t3) {
    const ct_pair64 x = ct_swap32(t0, t2), y = ct_swap32(t1, t3);
    const double a = x.a + x.b, b = y.a + y.b;
    const auto l = __builtin_amdgcn_permlane16_swap(ct_lo(a), ct_lo(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ct_hi(a), ct_hi(b), false, false);
    return ct_join(l[0], h[0]) + ct_join(l[1], h[1]);
}

// The tridiagonalization in fp64, for fp32 factors (ct_tridiagonalize64 says
// why). G: the fp32 Gram matrices, iu[v] the scale of half v. dv, ev: element c
// of T's diagonal and off-diagonal.
__device__ __forceinline__ void c16_tridiagonalize64(const cq_f32x16 &G, const float (&iu)[4], float *sV, double *sU,
                                                     float &dv, float &ev) {
    constexpr int P = 16;
    const int lane = threadIdx.x, c = lane & 15, b = lane >> 4;
    ct_f64x16 D;
#pragma unroll
    for (int i = 0; i < 16; ++i) D[i] = (double)G[i] * (double)iu[i >> 2];
    auto row = [&](int k) -> double {
        const int i = k & 3;
        const ct_pair64 x = ct_swap32(D[i], D[8 + i]), y = ct_swap32(D[4 + i], D[12 + i]);
        const double p = (k & 8) ? x.b : x.a, q = (k & 8) ? y.b : y.a;
        const auto l = __builtin_amdgcn_permlane16_swap(ct_lo(p), ct_lo(q), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ct_hi(p), ct_hi(q), false, false);
        return (k & 4) ? ct_join(l[1], h[1]) : ct_join(l[0], h[0]);
    };
    double tri_d = 0.0, tri_e = 0.0;
#pragma unroll 1
    for (int k = 0; k < P - 2; ++k) {
        const double rw = row(k);
        const double x1 = __shfl(rw, (lane & 48) + k + 1, 64);
        const double x = c > k ? rw : 0.0;
        const double s2 = ct_sum<16>(x * x);
        const double alpha = s2 > 1e-60 ? -__builtin_copysign(s2 * ct_rsq(s2), x1) : 0.0;
        tri_d = c == k ? rw : tri_d;
        tri_e = c == k ? alpha : tri_e;
        const double hh = fma(fabs(x1), fabs(alpha), s2);
        const double y = hh > 1e-36 ? ct_rsq(hh) : 0.0;
        const double u = (c == k + 1 ? x1 - alpha : x) * y;
        sV[(b * 14 + k) * 16 + c] = (float)u;
        sU[lane] = u;
        ct_lds_fence();
        double t[4];
        ct_f64x4 ub[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            ub[v] = ct_ld4(sU + 16 * v + 4 * b);   // rows 4 q .. of half v
            t[v] = fma(D[4 * v], ub[v][0], fma(D[4 * v + 1], ub[v][1], fma(D[4 * v + 2], ub[v][2], D[4 * v + 3] * ub[v][3])));
        }
        const double p = c > k ? c16_row_sums(t[0], t[1], t[2], t[3]) : 0.0;
        const double w = fma(-0.5 * ct_sum<16>(p * u), u, p);
        sU[64 + lane] = w;
        ct_lds_fence();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const ct_f64x4 wb = ct_ld4(sU + 64 + 16 * v + 4 * b);
            const double uc = sU[16 * v + c], wc = sU[64 + 16 * v + c];
#pragma unroll
            for (int i = 0; i < 4; ++i) D[4 * v + i] = fma(-wb[i], uc, fma(-ub[v][i], wc, D[4 * v + i]));
        }
        ct_lds_fence();
    }
    const double r0 = row(P - 2), r1 = row(P - 1);
    const double e0 = __shfl(r0, (lane & 48) + P - 1, 64);
    dv = (float)(c == P - 2 ? r0 : c == P - 1 ? r1 : tri_d);
    ev = (float)(c == P - 2 ? e0 : c == P - 1 ? 0.0 : tri_e);
}

template <typename TF, bool kList>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
void k_compress_tri16(Geo g, pkv_page *table, const char *dense, char *factor, CompressItems items, CompressSrc src,
                      int64_t n_items) {
    constexpr int P = 16;
    constexpr bool kF64 = ct_f64<TF>();
    __shared__ __align__(32) float smem[c16_lds(kF64)];
    const int d = g.d;
    const int lane = threadIdx.x, c = lane & 15, b = lane >> 4;   // element c of half b; also column n and rows 4 q
    float *sV = smem;                        // reflector k of half b at (b * 14 + k) * 16
    float *sQ = sV + 4 * 14 * 16;            // d_0, e_0, d_1, e_1, ... per half
    float2 *sT = (float2 *)(sQ + 128);       // (d_i, e_{i-1}^2) per half
    float *sZ = smem;

    const int64_t item0 = 2 * (int64_t)blockIdx.x;
    bool active[2];
    int64_t entry[2];
    int rank[4];
    const uint16_t *X[4];
    bool tr[4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const DecompRef ref = decode_decomp<uint16_t, kList>(g, table, dense, items, src, 2 * (item0 + t) + w,
                                                                 2 * n_items, lane == 0 && w == 0);
            active[t] = ref.active;
            entry[t] = ct_scalar(ref.active ? g.head_index(ref.b, ref.h) * g.max_pages + ref.j : 0);
            rank[2 * t + w] = w == 0 ? ref.rk : ref.rv;
            X[2 * t + w] = (const uint16_t *)ct_scalar((int64_t)ref.X);
            tr[2 * t + w] = ref.transposed;
        }
    }
    if (!active[0] && !active[1]) return;
    // a page that is out of range or refused: its half of the wavefront redoes the other page, unstored
#pragma unroll
    for (int t = 0; t < 2; ++t)
        if (!active[t])
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                X[2 * t + w] = X[2 - 2 * t + w];
                tr[2 * t + w] = tr[2 - 2 * t + w];
                rank[2 * t + w] = rank[2 - 2 * t + w];
            }

    // ---- 1. Gram matrices (rows of a page are read as 16-byte operands) ---------
    cq_f32x16 G;
    float fro2 = 0.f;   // |G|_F^2 of half b
    {
        c16_f32x4 acc[4] = {};
        for (int s = 0; s < d / 32; ++s)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const cq_bf16x8 a = cq_load8(X[u], tr[u], P, d, c, 32 * s + 8 * b);
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, a, acc[u], 0, 0, 0);
            }
        float f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            f[u] = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                G[4 * u + i] = acc[u][i];
                f[u] = fmaf(acc[u][i], acc[u][i], f[u]);
            }
        }
        fro2 = ct_sum<16>(c16_row_sums(f[0], f[1], f[2], f[3]));
    }
    const float gnorm = sqrtf(fro2);
    float iu[4];   // 1 / |G|_F of every half
#pragma unroll
    for (int u = 0; u < 4; ++u) iu[u] = cq_f(__builtin_amdgcn_readlane(cq_i(gnorm > 0.f ? 1.f / gnorm : 0.f), 16 * u));

    // ---- 2. tridiagonalization -----------------------------------------------------
    float dv = 0.f, ev = 0.f;   // T's diagonal and, below it, its off-diagonal, element c
    if constexpr (kF64) {
        c16_tridiagonalize64(G, iu, sV, (double *)(sQ + 256), dv, ev);
    } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) G[i] *= iu[i >> 2];
    // row k of every half, one element per lane: from lane row k / 4
    auto row = [&](int k) -> float {
        const int i = k & 3;
        const ct_pair x = ct_swap32(G[i], G[8 + i]), y = ct_swap32(G[4 + i], G[12 + i]);
        const ct_pair s = (k & 8) ? c16_swap16(x.b, y.b) : c16_swap16(x.a, y.a);
        return (k & 4) ? s.b : s.a;
    };
    for (int k = 0; k < P - 2; ++k) {
        const float rw = row(k);
        const float x1 = __shfl(rw, (lane & 48) + k + 1, 64);
        const float x = c > k ? rw : 0.f;
        const float s2 = ct_sum<16>(x * x);
        const float alpha = -__builtin_copysignf(__builtin_amdgcn_sqrtf(s2), x1);
        dv = c == k ? rw : dv;
        ev = c == k ? alpha : ev;
        const float hh = fmaf(fabsf(x1), fabsf(alpha), s2);
        float y = __builtin_amdgcn_rsqf(hh);
        y *= fmaf(-0.5f * hh * y, y, 1.5f);
        y = hh > 1e-36f ? y : 0.f;
        const float u = (c == k + 1 ? x1 - alpha : x) * y;
        sV[(b * 14 + k) * 16 + c] = u;
        ct_lds_fence();
        float t[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float4 ub = *(const float4 *)(sV + (v * 14 + k) * 16 + 4 * b);   // rows 4 q .. of half v
            t[v] = fmaf(G[4 * v], ub.x, fmaf(G[4 * v + 1], ub.y, fmaf(G[4 * v + 2], ub.z, G[4 * v + 3] * ub.w)));
        }
        const float p = c > k ? c16_row_sums(t[0], t[1], t[2], t[3]) : 0.f;
        const float w = fmaf(-0.5f * ct_sum<16>(p * u), u, p);
        G = c16_outer(u, -w, G);
        G = c16_outer(w, -u, G);
    }
    const float r0 = row(P - 2), r1 = row(P - 1);
    const float e0 = __shfl(r0, (lane & 48) + P - 1, 64);
    dv = c == P - 2 ? r0 : c == P - 1 ? r1 : dv;
    ev = c == P - 2 ? e0 : c == P - 1 ? 0.f : ev;
    }   // fp32
    {
        const float before = __shfl(ev, (lane & 48) + ((c + 15) & 15), 64);   // e_{c-1}; e_{15} = 0
        ((float2 *)sQ)[lane] = make_float2(dv, ev);
        sT[lane] = make_float2(dv, fmaxf(before * before, 1e-36f));
    }
    ct_lds_fence();

    // ---- 3. the largest eigenvalues --------------------------------------------------
    const int r_most = max(max(rank[0], rank[1]), max(rank[2], rank[3]));
    const int r_own = b == 0 ? rank[0] : b == 1 ? rank[1] : b == 2 ? rank[2] : rank[3];
    const int lpe_log = r_most > 8 ? 0 : r_most > 4 ? 1 : 2, lpe = 1 << lpe_log;
    float lam;   // eigenvalue c >> lpe_log of half b
    {
        const float4 *td = (const float4 *)(sT + 16 * b);
        const int j = c >> lpe_log;
        auto count = [&](float x) {
            float q = 1.f;
            uint32_t bits = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float4 t = td[i];
                const float q0 = fmaf(-t.y, __builtin_amdgcn_rcpf(q), t.x - x);
                bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(q0), 31);
                q = fmaf(-t.w, __builtin_amdgcn_rcpf(q0), t.z - x);
                bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(q), 31);
            }
            return P - __popc(bits);
        };
        const int lo0 = __float_as_int(9.3132257e-10f), hi0 = __float_as_int(1.02f);
        constexpr int kStep = (0x3f828f5c - 0x30800000) / 16;
        const int cnt = count(__int_as_float(lo0 + kStep * c));
        int above = 0;
        for (int i = 0; i < r_most; ++i) {
            const int na = __popc((uint32_t)(__ballot(cnt > i) >> (lane & 48)) & 0xffffu);
            above = i == j ? na : above;
        }
        int lo = above > 0 ? lo0 + kStep * (above - 1) : 0;
        int hi = above < 16 ? lo0 + kStep * above : hi0;
        const float frac = (float)((c & (lpe - 1)) + 1) / (float)(lpe + 1);
        for (int it = 0; it < 32 && __any(j < r_own && hi - lo > ct_section_ulps(kF64) && lo > 0); ++it) {
            const int m = lo + (int)((float)(hi - lo) * frac);
            const bool up = count(__int_as_float(m)) > j;
            int nl = up ? m : lo, nh = up ? hi : m;
            for (int x = 1; x < lpe; x <<= 1) {
                nl = max(nl, __shfl_xor(nl, x, 64));
                nh = min(nh, __shfl_xor(nh, x, 64));
            }
            lo = nl;
            hi = max(nh, nl);
        }
        lam = __int_as_float(lo + ((hi - lo) >> 1));
    }

    // ---- 4. eigenvectors of T, two halves a pass: lane (direction, half, vector) -----
    // T from its last row up, as (d, e) pairs, in place of the (d, e^2) pairs
    ct_lds_fence();
    {
        const int cc = (lane & 48) + (P - 1 - c);
        const float e = c < P - 1 ? ((const float2 *)sQ)[cc - 1].y : 0.f;
        sT[lane] = make_float2(((const float2 *)sQ)[cc].x, e);
    }
    ct_lds_fence();
    uint32_t bad_half = 0;   // bit b: half b is left to k_compress
    float zt[2][P];          // rows of this lane's vector in its direction, per pass
    int meet[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int half = 2 * u + (b & 1);
        const int r = (b & 1) ? rank[2 * u + 1] : rank[2 * u];
        const float l = __shfl(lam, 16 * half + (min(c, r - 1) << lpe_log), 64);
        const float gn = __shfl(gnorm, 16 * half, 64);
        const float2 *Q = (const float2 *)sQ + 16 * half;
        int from = (b >> 1) * 128 + 32 * half;   // upper half of the wavefront: upwards
        asm volatile("" : "+v"(from));
        const float2 *H = (const float2 *)(sQ + from);
        float (&F)[P] = zt[u];
        {
            float ee = 0.f, rc = 0.f;
#pragma unroll
            for (int i = 0; i < P; ++i) {
                if (i % 8 == 0) ct_pace();
                const float2 t = H[i];
                const float f = fmaf(-ee * ee, rc, t.x - l);
                F[i] = __builtin_copysignf(fmaxf(fabsf(f), 1e-30f), f);
                ee = t.y;
                rc = __builtin_amdgcn_rcpf(F[i]);
            }
        }
        float best = INFINITY;
        int kk = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (i % 8 == 0) ct_pace();
            const float up = ct_swap32(F[P - 1 - i], F[P - 1 - i]).b;
            const float gi = fabsf(F[i] + (up - (Q[i].x - l)));
            kk = gi < best ? i : kk;
            best = fminf(gi, best);
        }
        kk = __float_as_int(ct_swap32(__int_as_float(kk), __int_as_float(kk)).a);
        best = ct_swap32(best, best).a;
        const int kl = b >= 2 ? P - 1 - kk : kk;
        const int klim = b >= 2 ? kl : kl + 1;   // the meeting row itself is the lower half's
        float zc = 1.f, nn = 0.f;
#pragma unroll
        for (int i = P - 1; i >= 0; --i) {
            if (i % 8 == 7) ct_pace();
            if (i + 1 < P) {
                asm volatile("" : "+v"(F[i]));
                const float t = -H[i].y * __builtin_amdgcn_rcpf(F[i]) * zc;
                zc = i < kl ? t : 1.f;
            }
            F[i] = i < klim ? zc : 0.f;
            nn = fmaf(F[i], F[i], nn);
        }
        {
            const ct_pair s = ct_swap32(nn, nn);
            nn = s.a + s.b;
        }
        const float inv = __builtin_amdgcn_rsqf(nn);
        const bool zero = gn == 0.f;   // a zero page: L the first unit vectors
        const bool bad = !zero && c < r && !(l > kCtTinyEig && best * inv <= kCtResidMax);
        const uint64_t m = __ballot(bad);
        bad_half |= ((m & 0x0000ffff0000ffffull) ? 1u : 0u) << (2 * u) | ((m & 0xffff0000ffff0000ull) ? 2u : 0u) << (2 * u);
        meet[u] = klim;
#pragma unroll
        for (int i = 0; i < P; ++i) F[i] = zero ? (b < 2 && i == c && c < r ? 1.f : 0.f) : c < r ? F[i] * inv : 0.f;
        if (zero) meet[u] = b >= 2 ? 0 : P;
    }
    // ---- 5. L = Q Z, orthonormalized ----------------------------------------------------
    // to lane (n, q): rows 4 q + i of vector n of half v in register 4 v + i. The
    // reflectors stay in LDS until they are applied, so the vectors take a
    // buffer of their own
    __shared__ float sX[4 * 16 * 16];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int half = 2 * u + (b & 1);
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int rowi = b >= 2 ? P - 1 - i : i;
            if (i < meet[u]) sX[(half * 16 + rowi) * 16 + c] = zt[u][i];
        }
    }
    ct_lds_fence();
    cq_f32x16 Z;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < 4; ++i) Z[4 * v + i] = sX[(v * 16 + 4 * b + i) * 16 + c];
    for (int k = P - 3; k >= 0; --k) {
        float4 ub[4];
        float t[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            ub[v] = *(const float4 *)(sV + (v * 14 + k) * 16 + 4 * b);
            t[v] = fmaf(Z[4 * v], ub[v].x, fmaf(Z[4 * v + 1], ub[v].y, fmaf(Z[4 * v + 2], ub[v].z, Z[4 * v + 3] * ub[v].w)));
        }
        const float s = c16_row_sums(t[0], t[1], t[2], t[3]);
        const ct_pair e = c16_swap16(s, s);                            // rows 0 0 2 2 and 1 1 3 3
        const ct_pair s02 = ct_swap32(e.a, e.a), s13 = ct_swap32(e.b, e.b);
        const float st[4] = {s02.a, s13.a, s02.b, s13.b};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            Z[4 * v] = fmaf(-st[v], ub[v].x, Z[4 * v]);
            Z[4 * v + 1] = fmaf(-st[v], ub[v].y, Z[4 * v + 1]);
            Z[4 * v + 2] = fmaf(-st[v], ub[v].z, Z[4 * v + 2]);
            Z[4 * v + 3] = fmaf(-st[v], ub[v].w, Z[4 * v + 3]);
        }
    }
    // bf16 factors: where k_compress stops for them, 10 P 2^-23
    constexpr float kTol = std::is_same<TF, uint16_t>::value ? 1.9e-5f : 3e-7f;
    for (int it = 0;; ++it) {
        c16_f32x4 S[4];
        bool more = false, last = true;   // a half that needs this step, and one after it
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            S[v] = c16_f32x4{};
#pragma unroll
            for (int i = 0; i < 4; ++i) S[v] = c16_mfma4(Z[4 * v + i], Z[4 * v + i], S[v]);
            bool bad = false;
            float e = 0.f, f2 = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float ei = fabsf(S[v][i] - (4 * b + i == c && c < rank[v] ? 1.f : 0.f));
                bad = bad || !(ei <= kOrthMax);
                e = fmaxf(e, ei);
                f2 = fmaf(ei, ei, f2);
            }
            const Orth next = orth_next(!__any(bad), !__any(e > kTol), 0.75f * ct_sum<64>(f2) <= kTol, it);
            if (next == Orth::fail) {   // left to k_compress: the others go on without it
                bad_half |= 1u << v;
            } else if (((bad_half >> v) & 1u) == 0) {
                more = more || next != Orth::done;
                last = last && next != Orth::step;
            }
        }
        if (!more) break;
        ct_lds_fence();
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int i = 0; i < 4; ++i) sZ[(v * 16 + 4 * b + i) * kC16ZStride + c] = Z[4 * v + i];
        ct_lds_fence();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float4 l = *(const float4 *)(sZ + (v * 16 + c) * kC16ZStride + 4 * b);   // row c, vectors 4 q ..
            c16_f32x4 y = {};
            const float lv[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                y = c16_mfma4(lv[i], fmaf(-0.5f, S[v][i], 4 * b + i == c ? 1.5f : 0.f), y);
#pragma unroll
            for (int i = 0; i < 4; ++i) Z[4 * v + i] = y[i];
        }
        if (last) break;
    }

    if constexpr (kF64) {   // unit length
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double nn = 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) nn = fma((double)Z[4 * v + i], (double)Z[4 * v + i], nn);
            const ct_pair64 h = ct_swap32(nn, nn);
            nn = h.a + h.b;
            const auto lo = __builtin_amdgcn_permlane16_swap(ct_lo(nn), ct_lo(nn), false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(ct_hi(nn), ct_hi(nn), false, false);
            const double inv = c < rank[v] ? ct_rsq(ct_join(lo[0], hi[0]) + ct_join(lo[1], hi[1])) : 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) Z[4 * v + i] = (float)((double)Z[4 * v + i] * inv);
        }
    }
    // ---- 6. R = L^T X, stores --------------------------------------------------------------
    ct_lds_fence();
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < 4; ++i) sZ[(v * 16 + 4 * b + i) * kC16ZStride + c] = Z[4 * v + i];
    ct_lds_fence();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int t = v >> 1, which = v & 1;
        if (!active[t]) continue;
        if ((bad_half >> (2 * t)) & 3u) {   // to k_compress, both halves of the page
            if (lane == 0 && which == 0) mark_page(table + entry[t], 3u);
            continue;
        }
        const int rk = rank[2 * t], rv = rank[2 * t + 1], rk4 = r4(rk), rv4 = r4(rv);
        const FactorLayout fl = factor_layout(P, d, rk, rv);
        TF *Ak = (TF *)(factor + entry[t] * g.factor_slot_bytes);
        if (which == 0) {   // A_K = L_K (16 x r4(rk)), one contiguous block
            const int nq = rk4 / 4;
            if (lane < 16 * nq) {
                const int tok = lane / nq, a4 = lane - tok * nq;
                ct_st4(Ak + 4 * lane, *(const float4 *)(sZ + (v * 16 + tok) * kC16ZStride + 4 * a4));
            }
        } else if (c < rv) {   // A_V^T = L_V^T (rv x 16)
            ct_st4(Ak + fl.avt + c * P + 4 * b, make_float4(Z[4 * v], Z[4 * v + 1], Z[4 * v + 2], Z[4 * v + 3]));
        }
        const uint16_t *Xv = X[v];
        if constexpr (std::is_same<TF, float>::value) {
            for (int k = c; k < d; k += 16) {
                c16_f32x4 acc = {};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc = c16_mfma4(Z[4 * v + i], bf16_to_f32(Xv[tr[v] ? k * P + 4 * b + i : (4 * b + i) * d + k]), acc);
                if (which == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (4 * b + i < rk) Ak[fl.bk + (4 * b + i) * d + k] = acc[i];
                } else if (4 * b < rv4) {
                    ct_st4(Ak + fl.bvt + k * rv4 + 4 * b, make_float4(acc[0], acc[1], acc[2], acc[3]));
                }
            }
        } else {
            // L in three bf16 parts (all its bits) against the exact page; dims k and k + 1 per lane
            uint32_t hw[2], mw[2], lw[2];
            cq_split3(Z[4 * v], Z[4 * v + 1], hw[0], mw[0], lw[0]);
            cq_split3(Z[4 * v + 2], Z[4 * v + 3], hw[1], mw[1], lw[1]);
            const c16_s16x4 lmid = __builtin_bit_cast(c16_s16x4, make_uint2(mw[0], mw[1]));
            const c16_s16x4 lhi = __builtin_bit_cast(c16_s16x4, make_uint2(hw[0], hw[1]));
            const c16_s16x4 llo = __builtin_bit_cast(c16_s16x4, make_uint2(lw[0], lw[1]));
            for (int k = 2 * c; k < d; k += 32) {
                uint2 e, o;
                if (tr[v]) {
                    e = *(const uint2 *)(Xv + k * P + 4 * b);
                    o = *(const uint2 *)(Xv + (k + 1) * P + 4 * b);
                } else {
                    uint32_t w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[i] = *(const uint32_t *)(Xv + i * d + (uint32_t)(4 * b * d + k));
                    e = make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u));
                    o = make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u));
                }
                const c16_s16x4 be = __builtin_bit_cast(c16_s16x4, e), bo = __builtin_bit_cast(c16_s16x4, o);
                c16_f32x4 ae = {}, ao = {};
                ae = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lhi, be, ae, 0, 0, 0);
                ao = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lhi, bo, ao, 0, 0, 0);
                ae = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lmid, be, ae, 0, 0, 0);
                ao = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lmid, bo, ao, 0, 0, 0);
                ae = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(llo, be, ae, 0, 0, 0);
                ao = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(llo, bo, ao, 0, 0, 0);
                if (which == 0) {   // R_K, rk x d
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (4 * b + i < rk) *(uint32_t *)(Ak + fl.bk + (4 * b + i) * d + k) = cq_pack_bf16(ae[i], ao[i]);
                } else if (4 * b < rv4) {   // R_V^T, d x r4(rv)
                    ct_st4(Ak + fl.bvt + k * rv4 + 4 * b, make_float4(ae[0], ae[1], ae[2], ae[3]));
                    ct_st4(Ak + fl.bvt + (k + 1) * rv4 + 4 * b, make_float4(ao[0], ao[1], ao[2], ao[3]));
                }
            }
        }
    }
}

// 16-token pages of bf16 whose rows can be read 16 bytes at a time.
inline bool compress_tri16_supported(const LaunchCtx &L, const CompressSrc &src) {
    const Geo &g = L.geo;
    if (g.dense_dtype != PKV_BF16 || g.P != 16 || g.d % 32 || g.d > 256) return false;
    const uintptr_t at = src.mode == SRC_CACHE ? (uintptr_t)L.c->dense_pool : (uintptr_t)src.k | (uintptr_t)src.v;
    return at % 16 == 0;
}

template <typename TF, bool kList>
hipError_t launch_compress_tri16_t(const LaunchCtx &L, const CompressItems &items, const CompressSrc &src,
                                   int64_t n_items) {
    const LayerPtrs p = layer_ptrs(L);
    hipLaunchKernelGGL((k_compress_tri16<TF, kList>), dim3((unsigned)ceil_div(n_items, (int64_t)2)), dim3(64), 0, L.stream,
                       L.geo, p.table, p.dense, p.factor, items, src, n_items);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_compress_marked16<TF>(L, items, src, n_items);
}

hipError_t launch_compress_tri16(const LaunchCtx &L, const CompressItems &items, const CompressSrc &src,
                                 int64_t n_decomp) {
    const bool fb = L.geo.factor_dtype == PKV_BF16;
    if (src.list)
        return fb ? launch_compress_tri16_t<uint16_t, true>(L, items, src, n_decomp / 2)
                  : launch_compress_tri16_t<float, true>(L, items, src, n_decomp / 2);
    return fb ? launch_compress_tri16_t<uint16_t, false>(L, items, src, n_decomp / 2)
              : launch_compress_tri16_t<float, false>(L, items, src, n_decomp / 2);
}

}  // namespace pkv
