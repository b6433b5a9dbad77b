// Fixed-order merges of partial slots, as device functions: the merge kernels call them, and where the slots of a
// (b,h) are few the kernels that consume the merged rows call them themselves (every workgroup for itself, into LDS),
// which saves a launch.  A merge kernel of this size costs 5 ... 9 us on the device (launch, two or three dependent
// memory latencies) and about 2.5 us on the host; reading the slots again in every workgroup 1 ... 2 us.
#ifndef FLARE_MERGE_H
#define FLARE_MERGE_H

#include "flare_internal.h"

namespace flare {

struct f16_t { uint16_t bits; };   // raw IEEE fp16 bits (a type of its own so that the row helpers can overload)

// Slots that a consumer merges itself: few enough to be walked over in order, and no more bytes per (b,h) than a
// workgroup reads in a microsecond or two from its L2.  (With more, the slot-parallel merge kernels are faster.)
constexpr int kInlineSlots = 16;
constexpr size_t kInlineBytes = 80 * 1024;
inline bool merge_inline(const flare_shape &s, int parts)
{
    return parts <= kInlineSlots && (size_t)parts * s.M * (s.d + 2) * 4 <= kInlineBytes;
}

// ---- log-sum-exps of fp32 storage --------------------------------------------------------------
// log2 (l 2^m).  v_log_f32 cuts its result, half an ulp on average (3e-7 nats for a sum of 2^15), the same way for every
// latent and token, and dV is proportional to both weights: the exponent is split off, so that what is cut is below 2^-24,
// and put back with one rounding to nearest.
__device__ __forceinline__ float lse_log2(float m, float l, float &frac)
{
    frac = log2f(__builtin_amdgcn_frexp_mantf(l));
    return m + (float)__builtin_amdgcn_frexp_expf(l);
}
__device__ __forceinline__ float lse_nat(float m, float l)
{
    constexpr float kLn2Low = -1.904654299957768e-9f;   // ln 2 - kLn2
    float frac;
    const float whole = lse_log2(m, l, frac);
    return fmaf(whole, kLn2, fmaf(whole, kLn2Low, frac * kLn2));
}

// ---- encode: z and lse_enc of one (b,h) -------------------------------------------------------
struct MergeZ {
    const float *m_part, *l_part, *o_part;   // slot p of latent m at [(b*h) * parts + p][M]
    float *z, *lse_enc;                      // [b*h][M][d], [b*h][M]
    int parts;                               // 0: z is complete, there is nothing to merge
    bool f32;                                // fp32 storage
};

// D / 4 threads per latent own four columns each; the slots are folded in order behind one maximum (exact in any order),
// so the bits depend on the slot count only.  A slot with m = -inf is empty.  R rows (`step` apart) go together, and the
// slots come four at a time, everything of four requested before anything is used: with all of kInlineSlots in flight the decode
// kernels around this took every register (68 ... 122 without it), and where their workgroups no longer all fit on the chip, half
// as much time again (12 x 8 heads, 56656 tokens, 32 latents: 151 us, 105 us like this).
template <int D, int R, typename Put>
__device__ __forceinline__ void merge_z_row(const MergeZ &g, int bh, int M, int m1, int m0, int step, int j, const Put &put,
                                            bool write)
{
    constexpr int P = 4;
    float gm[R], l[R];
    float4 o[R];
    size_t s0[R];                                         // slot p of row r: s0[r] + p * M
#pragma unroll
    for (int r = 0; r < R; ++r) {
        s0[r] = (size_t)bh * g.parts * M + (R == 1 ? m0 : min(m0 + r * step, m1 - 1));
        gm[r] = -INFINITY;
        l[r] = 0.f;
        o[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (g.parts > P) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int p = 0; p < kInlineSlots; ++p) gm[r] = fmaxf(gm[r], g.m_part[s0[r] + (size_t)min(p, g.parts - 1) * M]);
    }
#pragma unroll 1
    for (int p0 = 0; p0 < g.parts; p0 += P) {
        float mp[R][P], lp[R][P];
        float4 oc[R][P];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const size_t slot = s0[r] + (size_t)min(p0 + i, g.parts - 1) * M;
                mp[r][i] = g.m_part[slot];
                lp[r][i] = g.l_part[slot];
                oc[r][i] = *reinterpret_cast<const float4 *>(g.o_part + slot * D + 4 * j);
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (g.parts <= P) gm[r] = fmaxf(fmaxf(mp[r][0], mp[r][1]), fmaxf(mp[r][2], mp[r][3]));
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const float w = (p0 + i >= g.parts || mp[r][i] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mp[r][i] - gm[r]);
                l[r] = fmaf(lp[r][i], w, l[r]);
                o[r].x = fmaf(oc[r][i].x, w, o[r].x);
                o[r].y = fmaf(oc[r][i].y, w, o[r].y);
                o[r].z = fmaf(oc[r][i].z, w, o[r].z);
                o[r].w = fmaf(oc[r][i].w, w, o[r].w);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = m0 + r * step;
        if (R > 1 && m >= m1) continue;
        const float inv = 1.f / l[r];
        const size_t idx = (size_t)bh * M + m;
        const float4 x = make_float4(o[r].x * inv, o[r].y * inv, o[r].z * inv, o[r].w * inv);
        put(m, j, x);
        if (write) {
            *reinterpret_cast<float4 *>(g.z + idx * D + 4 * j) = x;
            if (j == 0) g.lse_enc[idx] = g.f32 ? lse_nat(gm[r], l[r]) : (gm[r] + log2f(l[r])) * kLn2;
        }
    }
}
// Rows m0 .. m1 by the nt threads of a workgroup; put(m, j, x) gets columns 4 j ... of row m, and with `write` they go to global
// memory.
template <int D, int R, typename Put>
__device__ __forceinline__ void merge_z_rows(const MergeZ &g, int bh, int M, int m0, int m1, int tid, int nt,
                                             const Put &put, bool write)
{
    constexpr int L = D / 4;
#pragma unroll 1
    for (int m = m0 + tid / L; m < m1; m += R * (nt / L)) merge_z_row<D, R>(g, bh, M, m1, m, nt / L, tid % L, put, write);
}
// ---- the variant of the last backward kernels ---------------------------------------------------
// They exist with one and with two exponentials per score.
// One exponential: P~ = 2^S2 as it comes, without a normaliser (S2 <= lse_enc2[m] and S2 <= lse_dec2[n], so with
// both log-sum-exps of a (b,h) within +-span nothing overflows and every weight that matters is a normal
// number), P = P~ e_m with e_m = 2^-lse_enc2[m] and R = P~ w_n with w_n = 2^-lse_dec2[n]:
//   dS = P (a - eps) + R (c - delta) = P~ (e_m (a - eps_m) + w_n (c - delta_n)),   dV += (e_m dZ_m) P~.
// e_m is folded into dZ where its partials are merged, BEFORE dZ is rounded to bf16 and eps = <dZ, Z> is formed
// (bwd_one_exp_ok decides there, and the kernels that follow take dZ and eps as they find them), so that a and
// eps still see the same rounded values and the score products need no correction k-step; w_n is a per-token
// scalar.  Anything else (log-sum-exps beyond +-span, non-finite statistics) takes the two-exponential
// form with dZ as it is.
// ld_range[b*h][part] = (min, max) of lse_dec2 as the dZ kernels recorded it.
// Called by a whole workgroup of at most 16 waves, all of whose threads take part in the reads (one memory latency, not
// one per 64 values); one barrier inside; every thread returns the same answer.  red: 64 floats of LDS.
// span: kPlanSpan, or kSpan32 with fp32 storage; below zero: two exponentials whatever the statistics.
constexpr float kPlanSpan = 60.f;
// fp32 storage: the planes of a value or gradient x beside a factor 2^-span end at 2^-133, bf16's smallest number, which must
// not be seen beside x: x from 2^-69 = 2e-21 up with 40 log2 units.  (The one plane of 16-bit storage is good to 2^-66
// with 60.)
constexpr float kSpan32 = 40.f;
__device__ __forceinline__ bool is_nan(float x) { return (__float_as_uint(x) & 0x7fffffffu) > 0x7f800000u; }
__device__ __forceinline__ bool bwd_one_exp_ok(const float *__restrict__ ld_range, const float *__restrict__ lse_enc,
                                               int bh, int parts, int M, float span, float *red)
{
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
    // the largest of lse_enc2, -lse_enc2, lse_dec2, -lse_dec2
    float worst = -INFINITY;
    bool nan = false;
    for (int m = tid; m < M; m += nt) {
        const float v = lse_enc[(size_t)bh * M + m] * kLog2e;
        nan |= is_nan(v);
        worst = fmaxf(worst, fabsf(v));
    }
    for (int p = tid; p < parts; p += nt) {
        const float a = ld_range[2 * ((size_t)bh * parts + p)], b = ld_range[2 * ((size_t)bh * parts + p) + 1];
        nan |= is_nan(a) || is_nan(b);
        worst = fmaxf(worst, fmaxf(-a, b));
    }
    if (nan) worst = INFINITY;                       // a NaN anywhere makes the test fail
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) worst = fmaxf(worst, __shfl_xor(worst, off));
    if (lane == 0) red[wave] = worst;
    __syncthreads();
    for (int i = 0; i < nt / 64; ++i) worst = fmaxf(worst, red[i]);
    return worst <= span;
}

// ---- dZ and eps of one (b,h) ------------------------------------------------------------------
struct MergeDz {
    const float *part, *ld_range;   // slots as above; ranges of lse_dec2
    float *dz, *eps;                // [b*h][M][d], [b*h][M]
    int *plan;                      // [b*h]: 1 = one exponential
    int parts;                      // 0: dz, eps and plan are complete
    float span;                     // of bwd_one_exp_ok
    unsigned lds;                   // byte offset of the merged rows in the workgroup's dynamic LDS
};

__device__ __forceinline__ float bf16_rounded(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xffff0000u);
}
__device__ __forceinline__ void add4(float4 &a, const float4 &b)
{
    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
}
// Four columns of a row summed over at most P slots in slot order, all of them requested first; slot p at p + i * stride.
template <int P>
__device__ __forceinline__ float4 sum_slots_upto(const float *__restrict__ p, size_t stride, int n)
{
    float4 t[P], a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < P; ++i) t[i] = *reinterpret_cast<const float4 *>(p + (size_t)min(i, n - 1) * stride);
#pragma unroll
    for (int i = 0; i < P; ++i)
        if (i < n) add4(a, t[i]);
    return a;
}
// Row m (four columns, D / 4 lanes per row, called together) of dZ: the sum of its slots, and what else goes into it.
struct DzRow { float4 a, z; float lse_enc; };
template <int D>
__device__ __forceinline__ DzRow load_dz_row(const float *__restrict__ part, const float *__restrict__ z,
                                             const float *__restrict__ lse_enc, int bh, int M, int parts, int m, int j)
{
    const size_t idx = (size_t)bh * M + m, stride = (size_t)M * D;
    const float *p = part + ((size_t)bh * parts * M + m) * D + 4 * j;
    DzRow r;
    r.z = *reinterpret_cast<const float4 *>(z + idx * D + 4 * j);
    r.lse_enc = lse_enc[idx];
    r.a = parts <= 4 ? sum_slots_upto<4>(p, stride, parts) : parts <= 8 ? sum_slots_upto<8>(p, stride, parts)
                                                                 : sum_slots_upto<kInlineSlots>(p, stride, parts);
    return r;
}
// The row scaled and rounded as its consumers want it, and eps_m (in every lane of the row).
template <int D>
__device__ __forceinline__ float4 finish_dz_row(const DzRow &r, int j, bool one_exp, bool round_bf16, float &eps)
{
    constexpr int L = D / 4;
    float4 a = r.a;
    if (one_exp) {                                   // the one-exponential kernels take dZ scaled by 2^-lse_enc2[m]
        // (of fp32 storage without the rounding of le log2 e, up to 1e-6 of 2^20)
        const float em = round_bf16 ? exp2f(-r.lse_enc * kLog2e) : expf(-r.lse_enc);
        a = make_float4(a.x * em, a.y * em, a.z * em, a.w * em);
    }
    // The 16-bit kernels take dZ as a bf16 operand.  Rounding it here, before eps is formed, keeps
    // a[m][n] = <dZ_m, V_n - Z_m> an exact expression in the rounded dZ (eps and the products see the same
    // values), instead of leaving <V_n, rounding error> uncancelled in every score.
    if (round_bf16) a = make_float4(bf16_rounded(a.x), bf16_rounded(a.y), bf16_rounded(a.z), bf16_rounded(a.w));
    float e = fmaf(a.w, r.z.w, fmaf(a.z, r.z.z, fmaf(a.y, r.z.y, a.x * r.z.x)));
#pragma unroll
    for (int off = 1; off < L; off <<= 1) {          // fixed tree over the row's lanes (L is a power of two)
        const float o = __shfl_xor(e, off);
        e = ((j & off) == 0) ? (e + o) : (o + e);
    }
    eps = e;
    return a;
}
template <int D>
__device__ __forceinline__ float4 merge_dz_row(const float *__restrict__ part, const float *__restrict__ z,
                                               const float *__restrict__ lse_enc, int bh, int M, int parts, int m,
                                               int j, bool one_exp, bool round_bf16, float &eps)
{
    return finish_dz_row<D>(load_dz_row<D>(part, z, lse_enc, bh, M, parts, m, j), j, one_exp, round_bf16, eps);
}
// What a consuming workgroup needs of one (b,h): the variant, and rows of dZ and eps: merged into `lds` (M * D, then M
// floats; with `write` they and the plan also go to global memory, for a later kernel) or in global memory.  Ends with
// a barrier when it merges.  red: 64 floats of LDS.  meanwhile(): called once, after the slots were requested.
template <int D, typename Meanwhile>
__device__ __forceinline__ bool merged_dz(const MergeDz &g, const float *z, const float *lse_enc, int bh, int M,
                                          bool round_bf16, bool write, float *lds, float *red, const float *&dz,
                                          const float *&eps, const Meanwhile &meanwhile)
{
    dz = g.dz + (size_t)bh * M * D;
    eps = g.eps + (size_t)bh * M;
    if (g.parts == 0) {
        meanwhile();
        return g.plan[bh] != 0;
    }
    constexpr int L = D / 4;
    // R rows a thread go together, all of their slots requested before the variant is decided (its test waits for memory too)
    constexpr int R = D == 32 ? 2 : 1;
    const int j = threadIdx.x % L, rows = blockDim.x / L;
    DzRow r[R];
    auto load = [&](int m0) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            r[i] = load_dz_row<D>(g.part, z, lse_enc, bh, M, g.parts, min(m0 + i * rows + (int)threadIdx.x / L, M - 1), j);
    };
    load(0);
    meanwhile();
    const bool one = bwd_one_exp_ok(g.ld_range, lse_enc, bh, g.parts, M, g.span, red);
    for (int m0 = 0; m0 < M; m0 += R * rows) {       // whole rows of lanes stay together (shuffles)
        if (m0 > 0) load(m0);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int m = m0 + i * rows + threadIdx.x / L;
            float e;
            const float4 a = finish_dz_row<D>(r[i], j, one, round_bf16, e);
            if (m < M) {
                *reinterpret_cast<float4 *>(lds + (size_t)m * D + 4 * j) = a;
                if (j == 0) lds[(size_t)M * D + m] = e;
                if (write) {
                    *reinterpret_cast<float4 *>(g.dz + ((size_t)bh * M + m) * D + 4 * j) = a;
                    if (j == 0) g.eps[(size_t)bh * M + m] = e;
                }
            }
        }
    }
    if (write && threadIdx.x == 0) g.plan[bh] = one ? 1 : 0;
    __syncthreads();
    dz = lds;
    eps = lds + (size_t)M * D;
    return one;
}

// ---- dQ ---------------------------------------------------------------------------------------
// four neighbouring elements of a row
__device__ __forceinline__ void store_four(float *p, const float4 &a) { *reinterpret_cast<float4 *>(p) = a; }
__device__ __forceinline__ void store_four(uint16_t *p, const float4 &a)   // bf16
{
    *reinterpret_cast<uint2 *>(p) =
        make_uint2((__float_as_uint(bf16_rounded(a.x)) >> 16) | __float_as_uint(bf16_rounded(a.y)),
                   (__float_as_uint(bf16_rounded(a.z)) >> 16) | __float_as_uint(bf16_rounded(a.w)));
}
__device__ __forceinline__ void store_four(f16_t *p, const float4 &a)
{
    typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
    half4_t t;
    t[0] = (_Float16)a.x; t[1] = (_Float16)a.y; t[2] = (_Float16)a.z; t[3] = (_Float16)a.w;
    *reinterpret_cast<half4_t *>(p) = t;
}

}  // namespace flare

#endif  // FLARE_MERGE_H
