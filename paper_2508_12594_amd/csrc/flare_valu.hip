// fp32 vector-ALU kernels of the FLARE mixer for the 16-bit shapes that the matrix-core kernels do not take (more than
// 2048 latents, fewer than 16 tokens), the kernels that merge partial sums for every path, and the backward's sequence
// of launches.
//
// Two kernel shapes cover every step of the vector path:
//   * one thread per LATENT, streaming tokens (encode partials, dZ partials, dQ partials):
//     the token rows k_n, v_n, dy_n have wave-uniform addresses, so they arrive through the
//     scalar data path (reads only) and cost no vector memory traffic or LDS;
//   * one thread per TOKEN, streaming latents (decode, token statistics, dK/dV): here
//     q_m, z_m, dZ_m are the wave-uniform operands.
// Scores are kept in log2 units, S2 = (scale*log2 e) * <q,k>, so that the softmax needs
// one v_exp_f32 per score.  Every cross-block reduction goes through per-chunk partials
// that are merged in a fixed order: results are bit-reproducible.
//
// Equations: Section 3.1, Eq. flare_encode / Eq. flare_decode; Appendix F per-latent and
// per-token forms.  The backward follows the formulas in include/flare.h.
#include <stdlib.h>

#include <type_traits>

#include "flare_internal.h"
#include "flare_merge.h"

namespace flare {
namespace {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Load one row of D elements as floats.  `p` points at the first element of the row.
template <int D>
__device__ __forceinline__ void load_row(const float *__restrict__ p, float (&out)[D])
{
    const float4 *p4 = reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int i = 0; i < D / 4; ++i) {
        float4 t = p4[i];
        out[4 * i + 0] = t.x; out[4 * i + 1] = t.y; out[4 * i + 2] = t.z; out[4 * i + 3] = t.w;
    }
}
template <int D>
__device__ __forceinline__ void load_row(const bf16_t *__restrict__ p, float (&out)[D])
{
    if constexpr (D == 4) {
        uint2 t = *reinterpret_cast<const uint2 *>(p);
        out[0] = bf16_lo(t.x); out[1] = bf16_hi(t.x); out[2] = bf16_lo(t.y); out[3] = bf16_hi(t.y);
    } else {
        const uint4 *p4 = reinterpret_cast<const uint4 *>(p);
#pragma unroll
        for (int i = 0; i < D / 8; ++i) {
            uint4 t = p4[i];
            out[8 * i + 0] = bf16_lo(t.x); out[8 * i + 1] = bf16_hi(t.x);
            out[8 * i + 2] = bf16_lo(t.y); out[8 * i + 3] = bf16_hi(t.y);
            out[8 * i + 4] = bf16_lo(t.z); out[8 * i + 5] = bf16_hi(t.z);
            out[8 * i + 6] = bf16_lo(t.w); out[8 * i + 7] = bf16_hi(t.w);
        }
    }
}
template <int D>
__device__ __forceinline__ void load_row(const f16_t *__restrict__ p, float (&out)[D])
{
    const _Float16 *h = reinterpret_cast<const _Float16 *>(p);
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < D / 4; ++i) {
        const half4 t = *reinterpret_cast<const half4 *>(h + 4 * i);
        out[4 * i] = (float)t[0]; out[4 * i + 1] = (float)t[1]; out[4 * i + 2] = (float)t[2]; out[4 * i + 3] = (float)t[3];
    }
}
template <int D>
__device__ __forceinline__ void store_row(f16_t *__restrict__ p, const float (&in)[D])
{
    _Float16 *h = reinterpret_cast<_Float16 *>(p);
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < D / 4; ++i) {
        half4 t;
        t[0] = (_Float16)in[4 * i]; t[1] = (_Float16)in[4 * i + 1]; t[2] = (_Float16)in[4 * i + 2]; t[3] = (_Float16)in[4 * i + 3];
        *reinterpret_cast<half4 *>(h + 4 * i) = t;
    }
}
template <int D>
__device__ __forceinline__ void store_row(float *__restrict__ p, const float (&in)[D])
{
    float4 *p4 = reinterpret_cast<float4 *>(p);
#pragma unroll
    for (int i = 0; i < D / 4; ++i) p4[i] = make_float4(in[4 * i], in[4 * i + 1], in[4 * i + 2], in[4 * i + 3]);
}
template <int D>
__device__ __forceinline__ void store_row(bf16_t *__restrict__ p, const float (&in)[D])
{
    uint32_t w[D / 2];
#pragma unroll
    for (int i = 0; i < D / 2; ++i) w[i] = f32_to_bf16_rne(in[2 * i]) | (f32_to_bf16_rne(in[2 * i + 1]) << 16);
    if constexpr (D == 4) {
        *reinterpret_cast<uint2 *>(p) = make_uint2(w[0], w[1]);
    } else {
        uint4 *p4 = reinterpret_cast<uint4 *>(p);
#pragma unroll
        for (int i = 0; i < D / 8; ++i) p4[i] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
    }
}
template <int D>
__device__ __forceinline__ float dot(const float (&a)[D], const float (&b)[D])
{
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D; ++j) s = fmaf(a[j], b[j], s);
    return s;
}

// The thread-per-latent kernels read the token rows through the scalar data path (the address is the same for the
// whole wave), a handful of rows per request, and a wave can use none of them before all have arrived: with the
// rows coming from HBM every group of tokens costs several full memory latencies.  So each group first touches
// the rows of a later group with one vector load that needs no register: its data goes to a few bytes of LDS
// that nobody reads (global_load_lds_dword), and the rows are in the L2 when the scalar requests come.
// Lanes 8 i + t of every 32 touch row t of the group kPrefetchTokens on in tensor i (a, b, c; i = 3: a again).
// The tensors' addresses come in a second time as plain integers (RowTouch): a pointer derived from the kernel's
// own tensor arguments would make the compiler treat the rows as possibly overwritten by this load and take
// them off the scalar data path.
constexpr int kPrefetchTokens = 16;   // two groups of kGroup ahead
struct RowTouch {
    unsigned long long a, b, c;   // addresses of up to three token tensors (element (0,0,0,0)); unused: a again
    unsigned long long f, g;      // addresses of up to two per-token fp32 arrays [b*h][N] (lanes 24-27); or 0
};
template <typename T>
__device__ __forceinline__ void touch_rows(const RowTouch &rt, size_t base, const TokStride &ts, int n, int N,
                                           float *sink)
{
    const int lane = threadIdx.x & 31;
    const int tok = min(n + kPrefetchTokens + (lane & 7), N - 1);
    const unsigned long long which = (lane & 16) ? ((lane & 8) ? rt.a : rt.c) : ((lane & 8) ? rt.b : rt.a);
    const void *src = reinterpret_cast<const T *>(which) + base + tok_off(ts, tok);
    if (lane >= 24 && lane < 28 && rt.f != 0) {   // the statistics of tokens n + kPrefetchTokens and 32 further on
        const unsigned long long arr = (lane & 2) ? rt.g : rt.f;
        src = reinterpret_cast<const float *>(arr) + (size_t)blockIdx.y * N + min(n + kPrefetchTokens + 32 * (lane & 1), N - 1);
    }
    __builtin_amdgcn_global_load_lds(src, sink, 4, 0, 0);
}

inline unsigned long long addr(const void *p) { return (unsigned long long)(uintptr_t)p; }

constexpr int kLatentBlock = 256;  // threads per block in the thread-per-latent kernels
constexpr int kTokenBlock = 256;   // threads per block in the thread-per-token kernels
constexpr int kGroup = 8;          // scores handled between two running-max updates

// ---------------------------------------------------------------------------------------
// Encode partials: thread = latent m, block = (chunk of tokens, b*h, block of latents).
// Online softmax over the chunk's tokens; writes (running max, sum, unnormalised O) per chunk.
// ---------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kLatentBlock) void encode_partial_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
    float *__restrict__ m_part, float *__restrict__ l_part, float *__restrict__ o_part,
    TokStride ts, int H, int N, int M, int chunk_len, int chunks, float c2, RowTouch touch)
{
    const int m = blockIdx.z * kLatentBlock + threadIdx.x;
    if (m >= M) return;
    const int bh = blockIdx.y, h = bh % H, chunk = blockIdx.x;
    float qm[D];
    load_row<D>(q + (size_t)h * ts.sq + (size_t)m * D, qm);
#pragma unroll
    for (int j = 0; j < D; ++j) qm[j] *= c2;
    const T *kb = k + tok_base(ts, bh, H);
    const T *vb = v + tok_base(ts, bh, H);
    const int n0 = chunk * chunk_len;
    const int n1 = min(N, n0 + chunk_len);

    float mr = -INFINITY, l = 0.f, o[D];
#pragma unroll
    for (int j = 0; j < D; ++j) o[j] = 0.f;

    __shared__ float sink[kLatentBlock];
    int n = n0;
    for (; n + kGroup <= n1; n += kGroup) {
        touch_rows<T>(touch, tok_base(ts, bh, H), ts, n, N, sink);
        float s[kGroup];
        float gm = mr;
#pragma unroll
        for (int t = 0; t < kGroup; ++t) {
            float kr[D];
            load_row<D>(kb + tok_off(ts, (n + t)), kr);
            s[t] = dot<D>(qm, kr);
            gm = fmaxf(gm, s[t]);
        }
        const float al = fast_exp2(mr - gm);   // mr = -inf on the first group: exp2(-inf) = 0
        mr = gm;
        l *= al;
#pragma unroll
        for (int j = 0; j < D; ++j) o[j] *= al;
#pragma unroll
        for (int t = 0; t < kGroup; ++t) {
            const float p = fast_exp2(s[t] - mr);
            l += p;
            float vr[D];
            load_row<D>(vb + tok_off(ts, (n + t)), vr);
#pragma unroll
            for (int j = 0; j < D; ++j) o[j] = fmaf(p, vr[j], o[j]);
        }
    }
    for (; n < n1; ++n) {
        float kr[D], vr[D];
        load_row<D>(kb + tok_off(ts, n), kr);
        const float s = dot<D>(qm, kr);
        const float gm = fmaxf(mr, s);
        const float al = fast_exp2(mr - gm);
        mr = gm;
        const float p = fast_exp2(s - mr);
        l = l * al + p;
        load_row<D>(vb + tok_off(ts, n), vr);
#pragma unroll
        for (int j = 0; j < D; ++j) o[j] = fmaf(p, vr[j], o[j] * al);
    }
    const size_t slot = ((size_t)bh * chunks + chunk) * M + m;
    m_part[slot] = mr;
    l_part[slot] = l;
    store_row<D>(o_part + slot * D, o);
}

// Merges of many partial slots: a workgroup takes merge_rows rows (latents) of one (b*h), its 256 threads sixteen groups of
// slots: group g adds the slots g, g + 16, ... in order, four columns a lane, so that sixteen lanes read 256 contiguous bytes of
// a slot, and a fixed tree adds the sixteen results (lanes 16 and 32 apart, then the four waves through LDS): the association
// order depends on the slot count only (bit-reproducible).  These launches are bound by two or three memory latencies, so they
// want many workgroups with few loads in a row each.  (With sixteen rows a workgroup, a thread holding whole rows that the
// tree moved through sixty-four shuffles and more: 8 heads, 256 latents, 64 slots, d = 32: encode 11.7 us, dZ 13.7, dQ 9.9.)
constexpr int kMergeGroups = 16;
constexpr int merge_rows(int d) { return 64 / d; }          // rows of a workgroup: 256 bytes of a slot
template <int D>
struct MergeLane {
    int m, j, g;      // row, lane's four columns 4 j ..., slot group
    bool live;
    MergeLane() = default;
    __device__ __forceinline__ MergeLane(int block, int M)
    {
        constexpr int L = D / 4;
        const int row = block * merge_rows(D) + (threadIdx.x & 15) / L;
        live = row < M;
        m = live ? row : M - 1;
        j = (threadIdx.x & 15) % L;
        g = threadIdx.x >> 4;
    }
};
struct MergeSum { float m, l; float4 o; };      // stabiliser, sum of weights, weighted columns
__device__ __forceinline__ MergeSum fold_pair(const MergeSum &a, const MergeSum &b)
{
    MergeSum r;
    r.m = fmaxf(a.m, b.m);
    const float wa = (a.m == -INFINITY) ? 0.f : fast_exp2(a.m - r.m);
    const float wb = (b.m == -INFINITY) ? 0.f : fast_exp2(b.m - r.m);
    r.l = a.l * wa + b.l * wb;
    r.o = make_float4(a.o.x * wa + b.o.x * wb, a.o.y * wa + b.o.y * wb, a.o.z * wa + b.o.z * wb, a.o.w * wa + b.o.w * wb);
    return r;
}
__device__ __forceinline__ float4 shfl_xor4(const float4 &x, int off)
{
    return make_float4(__shfl_xor(x.x, off), __shfl_xor(x.y, off), __shfl_xor(x.z, off), __shfl_xor(x.w, off));
}

// z and lse_enc of many encode slots.  A slot with m = -inf is empty and contributes nothing.
template <int D>
__global__ __launch_bounds__(256) void encode_merge_kernel(
    const float *__restrict__ m_part, const float *__restrict__ l_part, const float *__restrict__ o_part,
    float *__restrict__ z, float *__restrict__ lse_enc, int BH, int M, int parts, bool f32)
{
    // Neighbouring rows go to workgroups of one XCD (every eighth): m_part and l_part give a workgroup 8 to 32 bytes of a line of 128, which
    // each L2 would fetch for itself.  (8 heads, 100000 tokens, 2048 latents, d = 32: 35.5 -> 25.1 us, d = 16 24.7 -> 15.9; 512 latents
    // 12.5 -> 10.1.  The sums of dZ and dQ read whole lines only and gain nothing.)
    const int n = gridDim.x, xcd = blockIdx.x & 7;
    const MergeLane<D> at(xcd * (n >> 3) + min(xcd, n & 7) + (blockIdx.x >> 3), M);
    const int bh = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    MergeSum s{-INFINITY, 0.f, make_float4(0.f, 0.f, 0.f, 0.f)};
    // four slots at a time: their loads are all issued before the first is folded (one memory latency per batch)
    constexpr int kBatch = 4;
    for (int p0 = at.g; p0 < parts; p0 += kMergeGroups * kBatch) {
        MergeSum t[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int p = p0 + kMergeGroups * b;
            const size_t slot = ((size_t)bh * parts + min(p, parts - 1)) * M + at.m;
            t[b].m = p < parts ? m_part[slot] : -INFINITY;
            t[b].l = l_part[slot];
            t[b].o = *reinterpret_cast<const float4 *>(o_part + slot * D + 4 * at.j);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (t[b].m != -INFINITY) s = fold_pair(s, t[b]);
    }
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
        const MergeSum o{__shfl_xor(s.m, off), __shfl_xor(s.l, off), shfl_xor4(s.o, off)};
        s = (lane & off) == 0 ? fold_pair(s, o) : fold_pair(o, s);      // both lanes of a pair form the same sum
    }
    __shared__ MergeSum part[4][16];
    if (lane < 16) part[wave][lane] = s;
    __syncthreads();
    if (threadIdx.x >= 16 || !at.live) return;
    s = fold_pair(fold_pair(part[0][lane], part[1][lane]), fold_pair(part[2][lane], part[3][lane]));
    const float inv = 1.f / s.l;
    const size_t idx = (size_t)bh * M + at.m;
    *reinterpret_cast<float4 *>(z + idx * D + 4 * at.j) = make_float4(s.o.x * inv, s.o.y * inv, s.o.z * inv, s.o.w * inv);
    if (at.j == 0) lse_enc[idx] = f32 ? lse_nat(s.m, s.l) : (s.m + log2f(s.l)) * kLn2;
}

// The same merge for few partial slots (flare_merge.h).  With 16 threads per latent striding over the slots most of them
// would idle and each would fetch whole rows from scattered slots; here the D / 4 threads of a latent take the
// slots in order, so a workgroup reads one contiguous piece per slot.
constexpr int kFewSlots = 8;   // (measured: with 16 and 32 slots in a row the slot-parallel kernels are the faster ones)
template <int D>
__global__ __launch_bounds__(256) void encode_merge_few_kernel(const MergeZ g, int M)
{
    constexpr int ROWS = 256 / (D / 4);
    const int m0 = blockIdx.x * ROWS;
    merge_z_rows<D, 1>(g, blockIdx.y, M, m0, min(M, m0 + ROWS), threadIdx.x, 256, [](int, int, const float4 &) {}, true);
}

// ---------------------------------------------------------------------------------------
// Per-token pass over the latents.  MODE 0: decode, writes y.  MODE 1: backward statistics,
// writes lse_dec2[n] = log2 sum_m 2^S2[m][n] and delta[n] = <dY_n, Y_n>.
// ---------------------------------------------------------------------------------------
template <typename T, int D, int MODE>
__global__ __launch_bounds__(kTokenBlock) void token_pass_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const float *__restrict__ z,
    T *__restrict__ y, const T *__restrict__ dy, float *__restrict__ lse_dec2, float *__restrict__ delta,
    TokStride ts, int H, int N, int M, float c2, int y_f32)
{
    // y_f32 (MODE 0, 16-bit T): y points to fp32 rows (flare_shape.y_f32)
    const int n = blockIdx.x * kTokenBlock + threadIdx.x;
    const int bh = blockIdx.y, h = bh % H;
    const bool valid = n < N;
    const size_t row = (size_t)bh * N + (valid ? n : N - 1);                     // index of the per-token scalars
    const size_t trow = tok_base(ts, bh, H) + tok_off(ts, (valid ? n : N - 1));  // first element of the token's row
    float kn[D];
    load_row<D>(k + trow, kn);
#pragma unroll
    for (int j = 0; j < D; ++j) kn[j] *= c2;
    const T *qh = q + (size_t)h * ts.sq;
    const float *zb = z + (size_t)bh * M * D;

    float mr = -INFINITY, l = 0.f, acc[D];
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = 0.f;
    int m = 0;
    for (; m + kGroup <= M; m += kGroup) {
        float s[kGroup];
        float gm = mr;
#pragma unroll
        for (int t = 0; t < kGroup; ++t) {
            float qr[D];
            load_row<D>(qh + (size_t)(m + t) * D, qr);
            s[t] = dot<D>(kn, qr);
            gm = fmaxf(gm, s[t]);
        }
        const float al = fast_exp2(mr - gm);
        mr = gm;
        l *= al;
#pragma unroll
        for (int j = 0; j < D; ++j) acc[j] *= al;
#pragma unroll
        for (int t = 0; t < kGroup; ++t) {
            const float p = fast_exp2(s[t] - mr);
            l += p;
            float zr[D];
            load_row<D>(zb + (size_t)(m + t) * D, zr);
#pragma unroll
            for (int j = 0; j < D; ++j) acc[j] = fmaf(p, zr[j], acc[j]);
        }
    }
    for (; m < M; ++m) {
        float qr[D], zr[D];
        load_row<D>(qh + (size_t)m * D, qr);
        const float s = dot<D>(kn, qr);
        const float gm = fmaxf(mr, s);
        const float al = fast_exp2(mr - gm);
        mr = gm;
        const float p = fast_exp2(s - mr);
        l = l * al + p;
        load_row<D>(zb + (size_t)m * D, zr);
#pragma unroll
        for (int j = 0; j < D; ++j) acc[j] = fmaf(p, zr[j], acc[j] * al);
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] *= inv;
    if (!valid) return;
    if constexpr (MODE == 0) {
        if (sizeof(T) == 2 && y_f32) store_row<D>(reinterpret_cast<float *>(y) + trow, acc);
        else store_row<D>(y + trow, acc);
        if (lse_dec2) lse_dec2[row] = (mr + log2f(l)) * kLn2;   // optional saved statistic, natural log
    } else {
        float g[D];
        load_row<D>(dy + trow, g);
        lse_dec2[row] = mr + log2f(l);
        delta[row] = dot<D>(g, acc);
    }
}

// Token statistics of the backward from what the forward saved: delta[n] = <dY_n, Y_n> with the
// stored Y, lse_dec2[n] = lse_dec[n] * log2(e).  thread = one token row of one head, numbered in
// the memory order of the token tensors so that a wave reads consecutive rows; purely HBM-bound.
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(
    const T *__restrict__ y, const T *__restrict__ dy, const float *__restrict__ lse_dec,
    float *__restrict__ lse_dec2, float *__restrict__ delta, bool head_fastest, int H, int N, size_t rows)
{
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= rows) return;
    const size_t trow = t * D;     // both layouts are dense: row t of the tensor as it lies in memory
    size_t row = t;                // index into the [B][H][N] statistics
    if (head_fastest) {            // t = (b*N + n)*H + h
        const size_t bn = t / H, h = t % H, b = bn / N, n = bn % N;
        row = (b * H + h) * N + n;
    }
    float a[D], g[D];
    load_row<D>(y + trow, a);
    load_row<D>(dy + trow, g);
    delta[row] = dot<D>(a, g);
    lse_dec2[row] = lse_dec[row] * kLog2e;
}

// The same from the forward's fp32 y (flare_shape.y_f32): delta[n] = <dY_n, Y_n> with an unrounded Y.
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_y32_kernel(
    const float *__restrict__ y, const T *__restrict__ dy, float *__restrict__ delta, bool head_fastest, int H, int N,
    size_t rows)
{
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= rows) return;
    size_t row = t;
    if (head_fastest) {
        const size_t bn = t / H, h = t % H, b = bn / N, n = bn % N;
        row = (b * H + h) * N + n;
    }
    float a[D], g[D];
    load_row<D>(y + t * D, a);
    load_row<D>(dy + t * D, g);
    if constexpr (sizeof(T) == 2) {
        // The matrix-core kernels take dY as a bf16 operand (fp16 storage is rounded to bf16 when read), and
        // c - delta = <dY_n, Z_m - Y_n> only cancels if delta is formed from the same rounded values.
#pragma unroll
        for (int i = 0; i < D; ++i) {
            uint32_t u = __float_as_uint(g[i]);
            u += 0x7fffu + ((u >> 16) & 1u);
            g[i] = __uint_as_float(u & 0xffff0000u);
        }
    }
    delta[row] = dot<D>(a, g);
}

// ---------------------------------------------------------------------------------------
// dZ partials: thread = latent m; dZ[m] += R[n][m] dY[n] over the chunk's tokens.
// ---------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kLatentBlock) void dz_partial_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ dy,
    const float *__restrict__ lse_dec2, float *__restrict__ dz_part,
    TokStride ts, int H, int N, int M, int chunk_len, int chunks, float c2, RowTouch touch)
{
    const int m = blockIdx.z * kLatentBlock + threadIdx.x;
    if (m >= M) return;
    const int bh = blockIdx.y, h = bh % H, chunk = blockIdx.x;
    float qm[D];
    load_row<D>(q + (size_t)h * ts.sq + (size_t)m * D, qm);
#pragma unroll
    for (int j = 0; j < D; ++j) qm[j] *= c2;
    const T *kb = k + tok_base(ts, bh, H);
    const T *gb = dy + tok_base(ts, bh, H);
    const float *lb = lse_dec2 + (size_t)bh * N;
    const int n0 = chunk * chunk_len;
    const int n1 = min(N, n0 + chunk_len);
    float acc[D];
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = 0.f;
    __shared__ float sink[kLatentBlock];
    auto token = [&](int n) {
        float kr[D], g[D];
        load_row<D>(kb + tok_off(ts, n), kr);
        const float r = fast_exp2(dot<D>(qm, kr) - lb[n]);
        load_row<D>(gb + tok_off(ts, n), g);
#pragma unroll
        for (int j = 0; j < D; ++j) acc[j] = fmaf(r, g[j], acc[j]);
    };
    int n = n0;
    for (; n + kGroup <= n1; n += kGroup) {   // whole groups: the touch is unconditional, no branch inside the group
        touch_rows<T>(touch, tok_base(ts, bh, H), ts, n, N, sink);
#pragma unroll
        for (int t = 0; t < kGroup; ++t) token(n + t);
    }
    for (; n < n1; ++n) token(n);
    store_row<D>(dz_part + (((size_t)bh * chunks + chunk) * M + m) * D, acc);
}

// Fixed-order sum of many partial slots, shared by dZ and dQ (see encode_merge_kernel): the sums are in the first sixteen threads.
// Slot s of output row (outer, m) lives at  part[((s / inner) * n_outer + outer) * inner + s % inner][m]:
// dZ: outer = b*h, one group of `inner` slots;  dQ: outer = h, the slots of all batch items b (groups of `inner` partials
// each), i.e. the batch sum in b order.  One barrier inside.  R: row blocks of the workgroup, summed side by side.
template <int D, int R>
__device__ __forceinline__ void sum_slots(const float *__restrict__ part, int outer, int n_outer, int groups, int inner, int M,
                                          const MergeLane<D> (&at)[R], float4 (&acc)[R])
{
    __shared__ float4 waves[R][4][16];
    const int total = groups * inner, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    // four slots at a time: their loads are all issued before the first is added; the sums keep the slot order
    constexpr int kBatch = 4;
    for (int s0 = at[0].g; s0 < total; s0 += kMergeGroups * kBatch) {
        float4 t[R][kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int s = min(s0 + kMergeGroups * b, total - 1);
            const size_t slot = ((size_t)(s / inner) * n_outer + outer) * inner + (s % inner);
#pragma unroll
            for (int r = 0; r < R; ++r) t[r][b] = *reinterpret_cast<const float4 *>(part + (slot * M + at[r].m) * D + 4 * at[r].j);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (s0 + kMergeGroups * b < total)
#pragma unroll
                for (int r = 0; r < R; ++r) add4(acc[r], t[r][b]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) add4(acc[r], shfl_xor4(acc[r], off));
        if (lane < 16) waves[r][wave][lane] = acc[r];
    }
    __syncthreads();
    if (threadIdx.x < 16) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float4 a = waves[r][0][lane], b = waves[r][2][lane];
            add4(a, waves[r][1][lane]);
            add4(b, waves[r][3][lane]);
            add4(a, b);
            acc[r] = a;
        }
    }
}

// dZ[b*h][m] = sum of its partial slots; eps[m] = <dZ_m, Z_m>.  R row blocks a workgroup.
template <int D, int R>
__global__ __launch_bounds__(256) void dz_merge_kernel(
    const float *__restrict__ dz_part, const float *__restrict__ z,
    float *__restrict__ dz, float *__restrict__ eps, int BH, int M, int parts, int round_bf16,
    const float *__restrict__ ld_range, const float *__restrict__ lse_enc, int *__restrict__ plan, float span)
{
    MergeLane<D> at[R];
#pragma unroll
    for (int r = 0; r < R; ++r) at[r] = MergeLane<D>(blockIdx.x * R + r, M);
    const int bh = blockIdx.y;
    // matrix-core path: which variant of the next kernels runs for this (b,h) (every workgroup works it out for
    // itself: the one-exponential variant wants dZ scaled, see bwd_one_exp_ok); one more workgroup records it
    const bool record = plan != nullptr && blockIdx.x == gridDim.x - 1;
    DzRow row[R]{};
    if (!record) {
        if (threadIdx.x < 16) {                      // (with the slots: one memory latency)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const size_t idx = (size_t)bh * M + at[r].m;
                row[r].z = *reinterpret_cast<const float4 *>(z + idx * D + 4 * at[r].j);
                row[r].lse_enc = lse_enc[idx];
            }
        }
        float4 acc[R];
        sum_slots<D, R>(dz_part, bh, BH, 1, parts, M, at, acc);
#pragma unroll
        for (int r = 0; r < R; ++r) row[r].a = acc[r];
    }
    __shared__ float plan_red[64];
    const bool one_exp = plan != nullptr && bwd_one_exp_ok(ld_range, lse_enc, bh, parts, M, span, plan_red);
    if (record) {
        if (threadIdx.x == 0) plan[bh] = one_exp ? 1 : 0;
        return;
    }
    if (threadIdx.x >= 16) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const size_t idx = (size_t)bh * M + at[r].m;
        float e;
        const float4 a = finish_dz_row<D>(row[r], at[r].j, one_exp, round_bf16 != 0, e);
        if (!at[r].live) continue;
        *reinterpret_cast<float4 *>(dz + idx * D + 4 * at[r].j) = a;
        if (at[r].j == 0) eps[idx] = e;
    }
}

// Few slots: see encode_merge_few_kernel.
template <int D>
__global__ __launch_bounds__(256) void dz_merge_few_kernel(
    const float *__restrict__ dz_part, const float *__restrict__ z,
    float *__restrict__ dz, float *__restrict__ eps, int BH, int M, int parts, int round_bf16,
    const float *__restrict__ ld_range, const float *__restrict__ lse_enc, int *__restrict__ plan, float span)
{
    constexpr int L = D / 4, ROWS = 256 / L;
    const int j = threadIdx.x % L;
    const int m = blockIdx.x * ROWS + threadIdx.x / L;
    const int bh = blockIdx.y;
    __shared__ float plan_red[64];                   // as in dz_merge_kernel
    const bool one_exp = plan != nullptr && bwd_one_exp_ok(ld_range, lse_enc, bh, parts, M, span, plan_red);
    if (plan != nullptr && blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x == 0) plan[bh] = one_exp ? 1 : 0;
        return;
    }
    const int mc = min(m, M - 1);                    // no early exit: the row's lanes meet in shuffles
    float e;
    const float4 a = merge_dz_row<D>(dz_part, z, lse_enc, bh, M, parts, mc, j, one_exp, round_bf16 != 0, e);
    if (m >= M) return;
    *reinterpret_cast<float4 *>(dz + ((size_t)bh * M + m) * D + 4 * j) = a;
    if (j == 0) eps[(size_t)bh * M + m] = e;
}

// dq_lat in fp32, or (T: the storage type) rounded once as it is stored.
template <typename T, int D>
__global__ __launch_bounds__(256) void dq_reduce_few_kernel(
    const float *__restrict__ dq_part, T *__restrict__ dq, int B, int H, int M, int parts, float scale)
{
    constexpr int L = D / 4, ROWS = 256 / L;
    const int j = threadIdx.x % L;
    const int m = blockIdx.x * ROWS + threadIdx.x / L;
    const int h = blockIdx.y;
    if (m >= M) return;
    const int slots = B * parts;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int s = 0; s < kFewSlots; ++s)
        if (s < slots)
            add4(a, *reinterpret_cast<const float4 *>(
                        dq_part + ((((size_t)(s / parts) * H + h) * parts + s % parts) * M + m) * D + 4 * j));
    store_four(dq + ((size_t)h * M + m) * D + 4 * j, make_float4(a.x * scale, a.y * scale, a.z * scale, a.w * scale));
}

// ---------------------------------------------------------------------------------------
// dQ partials: thread = latent m;  dQ[m] += dS[m][n] k[n] over the chunk's tokens, with
// dS[m][n] = P[m][n](<dZ_m,V_n> - eps_m) + R[n][m](<dY_n,Z_m> - delta_n).
// ---------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kLatentBlock) void dq_partial_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dy,
    const float *__restrict__ z, const float *__restrict__ lse_enc, const float *__restrict__ dz,
    const float *__restrict__ eps, const float *__restrict__ lse_dec2, const float *__restrict__ delta,
    float *__restrict__ dq_part, TokStride ts, int H, int N, int M, int chunk_len, int chunks, float c2,
    RowTouch touch)
{
    const int m = blockIdx.z * kLatentBlock + threadIdx.x;
    if (m >= M) return;
    const int bh = blockIdx.y, h = bh % H, chunk = blockIdx.x;
    float qm[D], zm[D], dzm[D], acc[D];
    load_row<D>(q + (size_t)h * ts.sq + (size_t)m * D, qm);
    load_row<D>(z + ((size_t)bh * M + m) * D, zm);
    load_row<D>(dz + ((size_t)bh * M + m) * D, dzm);
#pragma unroll
    for (int j = 0; j < D; ++j) { qm[j] *= c2; acc[j] = 0.f; }
    const float le2 = lse_enc[(size_t)bh * M + m] * kLog2e;
    const float ep = eps[(size_t)bh * M + m];
    const T *kb = k + tok_base(ts, bh, H);
    const T *vb = v + tok_base(ts, bh, H);
    const T *gb = dy + tok_base(ts, bh, H);
    const float *lb = lse_dec2 + (size_t)bh * N;
    const float *db = delta + (size_t)bh * N;
    const int n0 = chunk * chunk_len;
    const int n1 = min(N, n0 + chunk_len);
    __shared__ float sink[kLatentBlock];
    auto token = [&](int n) {
        float kr[D], vr[D], g[D];
        load_row<D>(kb + tok_off(ts, n), kr);
        load_row<D>(vb + tok_off(ts, n), vr);
        load_row<D>(gb + tok_off(ts, n), g);
        const float s2 = dot<D>(qm, kr);
        const float p = fast_exp2(s2 - le2);
        const float r = fast_exp2(s2 - lb[n]);
        const float ds = p * (dot<D>(dzm, vr) - ep) + r * (dot<D>(zm, g) - db[n]);
#pragma unroll
        for (int j = 0; j < D; ++j) acc[j] = fmaf(ds, kr[j], acc[j]);
    };
    int n = n0;
    for (; n + kGroup <= n1; n += kGroup) {   // whole groups: the touch is unconditional, no branch inside the group
        touch_rows<T>(touch, tok_base(ts, bh, H), ts, n, N, sink);
#pragma unroll
        for (int t = 0; t < kGroup; ++t) token(n + t);
    }
    for (; n < n1; ++n) token(n);
    store_row<D>(dq_part + (((size_t)bh * chunks + chunk) * M + m) * D, acc);
}

// dq_lat[h][m] = scale * sum over batch items and partial slots (fixed order, see sum_slots).
template <typename T, int D>
__global__ __launch_bounds__(256) void dq_reduce_kernel(
    const float *__restrict__ dq_part, T *__restrict__ dq, int B, int H, int M, int parts, float scale)
{
    const MergeLane<D> at[1] = {MergeLane<D>(blockIdx.x, M)};
    const int h = blockIdx.y;
    float4 sum[1];
    sum_slots<D, 1>(dq_part, h, H, B, parts, M, at, sum);
    const float4 &a = sum[0];
    if (threadIdx.x < 16 && at[0].live)
        store_four(dq + ((size_t)h * M + at[0].m) * D + 4 * at[0].j, make_float4(a.x * scale, a.y * scale, a.z * scale, a.w * scale));
}

// ---------------------------------------------------------------------------------------
// dK, dV: thread = token n;  dK_n = scale * sum_m dS[m][n] q_m,  dV_n = sum_m P[m][n] dZ_m.
// ---------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(kTokenBlock) void dkdv_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dy,
    const float *__restrict__ z, const float *__restrict__ lse_enc, const float *__restrict__ dz,
    const float *__restrict__ eps, const float *__restrict__ lse_dec2, const float *__restrict__ delta,
    T *__restrict__ dk, T *__restrict__ dv, TokStride ts, int H, int N, int M, float scale)
{
    const int n = blockIdx.x * kTokenBlock + threadIdx.x;
    const int bh = blockIdx.y, h = bh % H;
    const bool valid = n < N;
    const size_t row = (size_t)bh * N + (valid ? n : N - 1);
    const size_t trow = tok_base(ts, bh, H) + tok_off(ts, (valid ? n : N - 1));
    const float c2 = scale * kLog2e;
    float kn[D], vn[D], g[D], ak[D], av[D];
    load_row<D>(k + trow, kn);
    load_row<D>(v + trow, vn);
    load_row<D>(dy + trow, g);
#pragma unroll
    for (int j = 0; j < D; ++j) { kn[j] *= c2; ak[j] = 0.f; av[j] = 0.f; }
    const float ld2 = lse_dec2[row];
    const float dl = delta[row];
    const T *qh = q + (size_t)h * ts.sq;
    const float *zb = z + (size_t)bh * M * D;
    const float *dzb = dz + (size_t)bh * M * D;
    const float *leb = lse_enc + (size_t)bh * M;
    const float *epb = eps + (size_t)bh * M;
    for (int m = 0; m < M; ++m) {
        float qr[D], zr[D], dzr[D];
        load_row<D>(qh + (size_t)m * D, qr);
        load_row<D>(zb + (size_t)m * D, zr);
        load_row<D>(dzb + (size_t)m * D, dzr);
        const float s2 = dot<D>(kn, qr);
        const float p = fast_exp2(s2 - leb[m] * kLog2e);
        const float r = fast_exp2(s2 - ld2);
        const float ds = p * (dot<D>(dzr, vn) - epb[m]) + r * (dot<D>(zr, g) - dl);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            ak[j] = fmaf(ds, qr[j], ak[j]);
            av[j] = fmaf(p, dzr[j], av[j]);
        }
    }
    if (!valid) return;
#pragma unroll
    for (int j = 0; j < D; ++j) ak[j] *= scale;
    store_row<D>(dk + trow, ak);
    store_row<D>(dv + trow, av);
}

// ---- workspace carving --------------------------------------------------------------------
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// dq_part: the dQ slots, where they may not share `part` with the dZ slots (kernels that merge those themselves)
struct BwdWs {
    float *lse_dec2, *delta, *part, *dz, *eps, *ld_range, *dq_part;
    int *plan;
    void *tok_part;
    float *acc32;
};

// Whether the kernels that need dZ merge its slots themselves.
inline bool dz_inline(const flare_shape &s)
{
    return s.dtype == FLARE_F32 ? mfma32_inline(s) : mfma_supported(s) && mfma_dz_inline(s);
}

// Partial slots per (b,h) of dZ and dQ, each region as long as its own kernels need.  (The vector kernels' 2048 / (b,h) slots,
// in both regions, made it up to 1.9 times as long: 3 x 16 heads, 2573 tokens, 104 latents, d = 32 54 MB, 11 like this.)
struct BwdSlots { int dz, dq; };
inline BwdSlots bwd_slots(const flare_shape &s, const ValuPlan &plan)
{
    if (!mfma_supported(s)) {
        flare_shape t = s;      // (what the caller is told to bring does not depend on the variant)
        t.variant = 0;
        const int blocks = s.dtype == FLARE_F32 ? mfma32_dq_blocks(t) : 0;
        return BwdSlots{plan.bwd.chunks, plan.bwd.chunks > blocks ? plan.bwd.chunks : blocks};
    }
    int dq = mfma_dq_fused(s) ? mfma_dkdv_blocks(s) : 0;
    // the dQ kernel's slots depend on the token order (dq_geom); what the caller is told to bring does not
    for (const flare_layout layout : {FLARE_BHND, FLARE_BNHD}) {
        flare_shape t = s;
        t.layout = layout;
        if (mfma_dq_parts(t) > dq) dq = mfma_dq_parts(t);
    }
    return BwdSlots{mfma_plan(s).parts, dq};
}

size_t bwd_layout(const flare_shape &s, const ValuPlan &plan, void *ws, BwdWs *out)
{
    const size_t BH = (size_t)s.B * s.H;
    const BwdSlots slots = bwd_slots(s, plan);
    const bool apart = dz_inline(s);   // else the dQ slots lie over those of dZ, merged by then
    size_t off = 0;
    char *base = static_cast<char *>(ws);
    if (out) out->lse_dec2 = reinterpret_cast<float *>(base + off);
    off += align256(BH * s.N * 4);
    if (out) out->delta = reinterpret_cast<float *>(base + off);
    off += align256(BH * s.N * 4);
    if (out) out->part = reinterpret_cast<float *>(base + off);
    off += align256(BH * (apart || slots.dz > slots.dq ? slots.dz : slots.dq) * s.M * s.d * 4);
    if (out) out->dz = reinterpret_cast<float *>(base + off);
    off += align256(BH * s.M * s.d * 4);
    if (out) out->eps = reinterpret_cast<float *>(base + off);
    off += align256(BH * s.M * 4);
    if (out) out->ld_range = reinterpret_cast<float *>(base + off);
    off += align256(BH * slots.dz * 2 * 4);
    if (out) out->plan = reinterpret_cast<int *>(base + off);
    off += align256(BH * 4);
    if (out) out->dq_part = out->part;
    if (apart) {
        if (out) out->dq_part = reinterpret_cast<float *>(base + off);
        off += align256(BH * slots.dq * s.M * s.d * 4);
    }
    if (mfma_supported(s)) {   // only shapes with more than 256 latents on the matrix-core path use these
        if (out) out->tok_part = base + off;
        off += mfma_tok_stats_bytes(s);
        if (out) out->acc32 = reinterpret_cast<float *>(base + off);
        off += mfma_dkdv_acc_bytes(s);
    } else if (out) {
        out->tok_part = nullptr;
        out->acc32 = nullptr;
    }
    return off;
}

inline int check_launch() { return hipGetLastError() == hipSuccess ? FLARE_OK : FLARE_ELAUNCH; }

template <typename T, int D>
int encode_impl(const flare_shape &s, const T *q, const T *k, const T *v, float *z, float *lse_enc,
                float scale, void *ws, hipStream_t stream)
{
    const ValuPlan plan = valu_plan(s);
    float *m_part, *l_part, *o_part;
    valu_fwd_layout(s, plan.enc, ws, &m_part, &l_part, &o_part);
    const int BH = s.B * s.H;
    const int lat_blocks = (s.M + kLatentBlock - 1) / kLatentBlock;
    if constexpr (std::is_same_v<T, float>) {
        const int rc = mfma32_encode(s, q, k, v, m_part, l_part, o_part, scale, stream);
        if (rc != FLARE_OK) return rc;
    } else {
        LaunchTimer t(KID_ENCODE_PARTIAL, stream);
        encode_partial_kernel<T, D><<<dim3(plan.enc.chunks, BH, lat_blocks), kLatentBlock, 0, stream>>>(
            q, k, v, m_part, l_part, o_part, tok_stride(s), s.H, s.N, s.M, plan.enc.chunk_len, plan.enc.chunks, scale * kLog2e,
            RowTouch{addr(k), addr(v), addr(k), 0, 0});
    }
    if (check_launch() != FLARE_OK) return FLARE_ELAUNCH;
    return launch_encode_merge(s, m_part, l_part, o_part, z, lse_enc, plan.enc.chunks, stream);
}

template <typename T, int D>
int decode_impl(const flare_shape &s, const T *q, const T *k, const float *z, T *y, float *lse_dec, float scale,
                hipStream_t stream)
{
    if constexpr (std::is_same_v<T, float>) {
        return mfma32_decode(s, q, k, z, y, lse_dec, scale, MergeZ{}, stream);
    } else {
        LaunchTimer t(KID_DECODE, stream);
        token_pass_kernel<T, D, 0><<<dim3((s.N + kTokenBlock - 1) / kTokenBlock, s.B * s.H), kTokenBlock, 0, stream>>>(
            q, k, z, y, nullptr, lse_dec, nullptr, tok_stride(s), s.H, s.N, s.M, scale * kLog2e, s.y_f32);
        return check_launch();
    }
}

// encode and decode; fp32 storage with few encode slots: the decode merges them itself
template <typename T, int D>
int forward_impl(const flare_shape &s, const T *q, const T *k, const T *v, T *y, float *z, float *lse_enc, float *lse_dec,
                 float scale, void *ws, hipStream_t stream)
{
    if constexpr (std::is_same_v<T, float>) {
        if (mfma32_inline(s)) {
            MergeZ g{nullptr, nullptr, nullptr, z, lse_enc, mfma32_split(s).chunks, true};
            float *m_part, *l_part, *o_part;
            valu_fwd_layout(s, mfma32_split(s), ws, &m_part, &l_part, &o_part);
            g.m_part = m_part;
            g.l_part = l_part;
            g.o_part = o_part;
            const int rc = mfma32_encode(s, q, k, v, m_part, l_part, o_part, scale, stream);
            return rc != FLARE_OK ? rc : mfma32_decode(s, q, k, z, y, lse_dec, scale, g, stream);
        }
    }
    const int rc = encode_impl<T, D>(s, q, k, v, z, lse_enc, scale, ws, stream);
    return rc != FLARE_OK ? rc : decode_impl<T, D>(s, q, k, z, y, lse_dec, scale, stream);
}

inline bool overlap(const void *a, const void *b, size_t bytes)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + bytes && y < x + bytes;
}

template <typename T, int D>
int backward_impl(const flare_shape &s, const T *q, const T *k, const T *v, const T *y, const float *lse_dec,
                  const T *dy, const float *z, const float *lse_enc, void *dq, bool dq_cast, T *dk, T *dv, float scale,
                  void *ws, hipStream_t stream)
{
    const ValuPlan plan = valu_plan(s);
    constexpr bool F32 = std::is_same_v<T, float>;   // matrix-core kernels of their own, for every shape
    const bool mf = mfma_supported(s);               // 16-bit storage: matrix-core kernels where they exist
    const bool planned = F32 || mf;                  // their kernels choose between one and two exponentials by (b,h)
    const int dz_parts = mf ? mfma_plan(s).parts : plan.bwd.chunks;
    BwdWs w;
    bwd_layout(s, plan, ws, &w);
    const int BH = s.B * s.H;
    const float c2 = scale * kLog2e;
    const TokStride ts = tok_stride(s);
    const int lat_blocks = (s.M + kLatentBlock - 1) / kLatentBlock;
    const dim3 tok_grid((s.N + kTokenBlock - 1) / kTokenBlock, BH);
    const dim3 lat_grid(plan.bwd.chunks, BH, lat_blocks);
    // token statistics: from what the forward saved, or recomputed.  On the matrix-core path the
    // saved ones need no pass of their own: the dZ kernel forms delta while it streams dY, and every
    // kernel reads lse_dec itself, scaled to log2 units.
    // With bf16 storage (or bf16 softmax weights behind fp16 storage: the matrix-core path) and d < 16,
    // delta = <dY_n, Y_n> from the forward's y is too coarse (few terms, and c - delta cancels): such
    // shapes recompute the statistics even when y and lse_dec are given.
    // The same with at most one tile of tokens: every dot product and sum is short, nothing averages the
    // rounding of y out (dq_lat, dK 2.1-2.4e-2 from the saved y, 8e-3 recomputed), and the recomputation costs
    // nothing at that size.
    // (at most one tile of tokens: any 16-bit y, also fp16 on the fp32 kernels)
    // Likewise with fewer tokens than latents: a latent's gradient is then a sum over few tokens (300 tokens, 1000
    // latents, d = 32: dq_lat 1.9e-2 ... 2.1e-2 from the saved y, 9e-3 recomputed).
    const bool bf16_weights = s.dtype == FLARE_BF16 || (s.dtype == FLARE_F16 && mf);
    const bool coarse_y = s.dtype != FLARE_F32 && ((bf16_weights && s.d < 16) || s.N <= 32 || s.N < s.M) &&
                          !(s.y_f32 && mf);   // an fp32 y is not coarse (the fp32 kernels, which take the
                                              // 16-bit shapes of fewer than 16 tokens, never read it: they recompute)
    const bool saved = y && lse_dec && !coarse_y;
    const bool fused = saved && planned;   // every later kernel is a matrix-core one
    const float *ld = fused ? lse_dec : w.lse_dec2;
    const float ld_mul = fused ? kLog2e : 1.f;
    // delta from the fp32 y: at d <= 8 inside the dZ kernel like from a 16-bit y, else by a pass of its own
    const bool y32 = fused && !F32 && s.y_f32 && s.d > 8;
    if constexpr (F32) {
        if (!saved) {
            const int rc = mfma32_token_stats(s, q, k, z, dy, w.lse_dec2, w.delta, scale, stream);
            if (rc != FLARE_OK) return rc;
        }
    } else if (y32) {
        LaunchTimer t(KID_BWD_PREP, stream);
        const size_t rows = (size_t)BH * s.N;
        bwd_prep_y32_kernel<T, D><<<(unsigned)((rows + 255) / 256), 256, 0, stream>>>(
            reinterpret_cast<const float *>(y), dy, w.delta, s.layout == FLARE_BNHD, s.H, s.N, rows);
    } else if (fused) {
    } else if (saved) {
        LaunchTimer t(KID_BWD_PREP, stream);
        const size_t rows = (size_t)BH * s.N;
        bwd_prep_kernel<T, D><<<(unsigned)((rows + 255) / 256), 256, 0, stream>>>(
            y, dy, lse_dec, w.lse_dec2, w.delta, s.layout == FLARE_BNHD, s.H, s.N, rows);
    } else if (mf) {
        const int rc = mfma_token_stats(s, q, k, z, dy, w.lse_dec2, w.delta, scale, w.tok_part, stream);
        if (rc != FLARE_OK) return rc;
    } else {
        LaunchTimer t(KID_BWD_TOKEN_STATS, stream);
        token_pass_kernel<T, D, 1><<<tok_grid, kTokenBlock, 0, stream>>>(q, k, z, nullptr, dy, w.lse_dec2, w.delta,
                                                                         ts, s.H, s.N, s.M, c2, 0);
    }
    if (check_launch() != FLARE_OK) return FLARE_ELAUNCH;
    if constexpr (F32) {
        const int rc = mfma32_dz_partial(s, q, k, dy, ld, ld_mul, fused ? y : nullptr, w.delta, w.ld_range, w.part, scale,
                                         stream);
        if (rc != FLARE_OK) return rc;
    } else if (mf) {
        int rc = mfma_dz_partial(s, q, k, dy, ld, ld_mul, (fused && !y32) ? y : nullptr,
                                 (fused && !y32) ? w.delta : nullptr, w.ld_range, w.part, scale, stream);
        if (rc != FLARE_OK) return rc;
    } else {
        {
            LaunchTimer t(KID_BWD_DZ_PARTIAL, stream);
            dz_partial_kernel<T, D><<<lat_grid, kLatentBlock, 0, stream>>>(q, k, dy, w.lse_dec2, w.part, ts, s.H,
                                                                           s.N, s.M, plan.bwd.chunk_len, plan.bwd.chunks,
                                                                           c2, RowTouch{addr(k), addr(dy), addr(k), addr(w.lse_dec2), addr(w.lse_dec2)});
        }
        if (check_launch() != FLARE_OK) return FLARE_ELAUNCH;
    }
    constexpr int kFewRows = 256 / (D / 4);   // rows per workgroup of the few-slot merge kernels
    const float span = (s.variant & FLARE_VARIANT_TWO_EXP) ? -1.f : F32 ? kSpan32 : kPlanSpan;   // bwd_one_exp_ok
    // A dQ kernel of its own runs before dK and dV are written, which may be over k, v or dy -- unless the dK/dV kernel
    // merges dZ for it.  Then it has to run behind that one, so dZ is merged first where the outputs lie over the inputs
    // (the same bits: merge_dz_row either way).
    const bool dq_fused = F32 ? mfma32_dq_fused(s) : mf && mfma_dq_fused(s);   // dQ comes out of the dK/dV kernel
    const size_t tok_bytes = (size_t)BH * s.N * D * sizeof(T);
    const bool in_place = overlap(dk, k, tok_bytes) || overlap(dk, v, tok_bytes) || overlap(dk, dy, tok_bytes) ||
                          overlap(dv, k, tok_bytes) || overlap(dv, v, tok_bytes) || overlap(dv, dy, tok_bytes);
    // what the dK/dV kernel has to merge itself, if anything
    const MergeDz merge{w.part, w.ld_range, w.dz, w.eps, w.plan, dz_inline(s) && (dq_fused || !in_place) ? dz_parts : 0,
                        span, 0u};
    if (merge.parts == 0) {
        LaunchTimer t(KID_BWD_DZ_MERGE, stream);
        if (dz_parts <= kFewSlots || dz_inline(s))
            dz_merge_few_kernel<D><<<dim3((s.M + kFewRows - 1) / kFewRows + (planned ? 1 : 0), BH), 256, 0, stream>>>(
                w.part, z, w.dz, w.eps, BH, s.M, dz_parts, mf ? 1 : 0, w.ld_range, lse_enc, planned ? w.plan : nullptr,
                span);
        else {
            // Two row blocks a workgroup where one each makes 2048 workgroups or more: each tests all of lse_enc for the variant, 8 KB of
            // L2 at 2048 latents beside 16 KB of slots.  (8 heads, 12000 tokens, 2000 latents, d = 16: 15.2 us by one, 11.7 by two, 12.8 by
            // four; d = 32 26.2, 20.2, 21.8; but 512 latents, d = 16 7.4, 7.9, 8.6.)
            const int blocks = (s.M + merge_rows(D) - 1) / merge_rows(D), two = (long long)blocks * BH >= 2048;
            const dim3 grid((two ? (blocks + 1) / 2 : blocks) + (planned ? 1 : 0), BH);
            auto kern = two ? dz_merge_kernel<D, 2> : dz_merge_kernel<D, 1>;
            kern<<<grid, 256, 0, stream>>>(w.part, z, w.dz, w.eps, BH, s.M, dz_parts, mf ? 1 : 0, w.ld_range, lse_enc,
                                           planned ? w.plan : nullptr, span);
        }
    }
    if (check_launch() != FLARE_OK) return FLARE_ELAUNCH;
    int dq_parts = plan.bwd.chunks;
    // shared latents: one gradient for all heads, summed over (b, h) in that fixed order
    const int groups = s.shared_latents ? BH : s.B, outers = s.shared_latents ? 1 : s.H;
    if (mf) dq_parts = dq_fused ? mfma_dkdv_blocks(s) : mfma_dq_parts(s);
    else if (dq_fused) dq_parts = mfma32_dq_blocks(s);
    auto dkdv = [&]() -> int {
        if constexpr (F32) {
            return mfma32_dkdv(s, q, k, v, dy, z, lse_enc, ld, w.delta, ld_mul, dk, dv, dq_fused ? w.dq_part : nullptr, scale,
                               merge, stream);
        } else if (mf) {
            const bool chunked = mfma_dkdv_acc_bytes(s) != 0;   // more than 256 latents: one pass per chunk
            int rc = FLARE_OK;
            for (int m0 = 0; m0 < s.M && rc == FLARE_OK; m0 += mfma_lat_step(s))   // each (b,h) slice by the variant its plan names
                rc = mfma_dkdv(s, q, k, v, dy, z, lse_enc, ld, w.delta, ld_mul, dk, dv, chunked ? w.acc32 : nullptr,
                               dq_fused ? w.dq_part : nullptr, m0, scale, merge, stream);
            return rc;
        } else {
            LaunchTimer t(KID_BWD_DKDV, stream);
            dkdv_kernel<T, D><<<tok_grid, kTokenBlock, 0, stream>>>(q, k, v, dy, z, lse_enc, w.dz, w.eps, w.lse_dec2,
                                                                    w.delta, dk, dv, ts, s.H, s.N, s.M, scale);
            return check_launch();
        }
    };
    auto dq_partials = [&]() -> int {
        if constexpr (F32) {
            return mfma32_dq_partial(s, q, k, v, dy, z, lse_enc, w.dz, w.eps, ld, w.delta, ld_mul, w.plan, w.dq_part, scale,
                                     stream);
        } else if (mf) {
            return mfma_dq_partial(s, q, k, v, dy, z, lse_enc, w.dz, w.eps, ld, w.delta, ld_mul, w.plan, w.dq_part, scale,
                                   stream);
        } else {
            LaunchTimer t(KID_BWD_DQ_PARTIAL, stream);
            dq_partial_kernel<T, D><<<lat_grid, kLatentBlock, 0, stream>>>(
                q, k, v, dy, z, lse_enc, w.dz, w.eps, w.lse_dec2, w.delta, w.dq_part, ts, s.H, s.N, s.M,
                plan.bwd.chunk_len, plan.bwd.chunks, c2, RowTouch{addr(k), addr(v), addr(dy), addr(w.lse_dec2), addr(w.delta)});
            return check_launch();
        }
    };
    int rc = FLARE_OK;
    if (!dq_fused && merge.parts == 0) rc = dq_partials();
    if (rc == FLARE_OK) rc = dkdv();
    if (!dq_fused && merge.parts != 0 && rc == FLARE_OK) rc = dq_partials();
    if (rc != FLARE_OK) return rc;
    auto reduce_dq = [&](auto *out) {
        typedef std::remove_reference_t<decltype(*out)> O;
        LaunchTimer t(KID_BWD_DQ_REDUCE, stream);
        if ((long long)groups * dq_parts <= kFewSlots)
            dq_reduce_few_kernel<O, D><<<dim3((s.M + kFewRows - 1) / kFewRows, outers), 256, 0, stream>>>(
                w.dq_part, out, groups, outers, s.M, dq_parts, scale);
        else
            dq_reduce_kernel<O, D><<<dim3((s.M + merge_rows(D) - 1) / merge_rows(D), outers), 256, 0, stream>>>(
                w.dq_part, out, groups, outers, s.M, dq_parts, scale);
    };
    if (dq_cast) reduce_dq(static_cast<T *>(dq));
    else reduce_dq(static_cast<float *>(dq));
    return check_launch();
}

// Dispatch on (dtype, d) to the template instances.
#define FLARE_DISPATCH(s, CALL)                                                   \
    do {                                                                          \
        if ((s).dtype == FLARE_F32) {                                             \
            typedef float T;                                                      \
            switch ((s).d) {                                                      \
                case 4: { constexpr int D = 4; return CALL; }                     \
                case 8: { constexpr int D = 8; return CALL; }                     \
                case 16: { constexpr int D = 16; return CALL; }                   \
                case 32: { constexpr int D = 32; return CALL; }                   \
            }                                                                     \
        } else if ((s).dtype == FLARE_F16) {                                      \
            typedef f16_t T;                                                      \
            switch ((s).d) {                                                      \
                case 4: { constexpr int D = 4; return CALL; }                     \
                case 8: { constexpr int D = 8; return CALL; }                     \
                case 16: { constexpr int D = 16; return CALL; }                   \
                case 32: { constexpr int D = 32; return CALL; }                   \
            }                                                                     \
        } else {                                                                  \
            typedef bf16_t T;                                                     \
            switch ((s).d) {                                                      \
                case 4: { constexpr int D = 4; return CALL; }                     \
                case 8: { constexpr int D = 8; return CALL; }                     \
                case 16: { constexpr int D = 16; return CALL; }                   \
                case 32: { constexpr int D = 32; return CALL; }                   \
            }                                                                     \
        }                                                                         \
        return FLARE_EUNSUPPORTED;                                                \
    } while (0)

}  // namespace

size_t valu_fwd_layout(const flare_shape &s, const Split &sp, void *ws, float **m_part, float **l_part,
                       float **o_part)
{
    const size_t slots = (size_t)s.B * s.H * sp.chunks * s.M;
    size_t off = 0;
    char *base = static_cast<char *>(ws);
    if (m_part) *m_part = reinterpret_cast<float *>(base + off);
    off += align256(slots * 4);
    if (l_part) *l_part = reinterpret_cast<float *>(base + off);
    off += align256(slots * 4);
    if (o_part) *o_part = reinterpret_cast<float *>(base + off);
    off += align256(slots * s.d * 4);
    return off;
}

int launch_encode_merge(const flare_shape &s, const float *m_part, const float *l_part, const float *o_part,
                        float *z, float *lse_enc, int parts, hipStream_t stream)
{
    const int BH = s.B * s.H;
    const dim3 blocks((s.M + merge_rows(s.d) - 1) / merge_rows(s.d), BH);
    LaunchTimer t(KID_ENCODE_MERGE, stream);
    if (parts <= kFewSlots || merge_inline(s, parts)) {   // (the same bits wherever a shape's slots are merged)
        const MergeZ g{m_part, l_part, o_part, z, lse_enc, parts, s.dtype == FLARE_F32};
#define FLARE_EMF(DD)                                                                                           \
    encode_merge_few_kernel<DD><<<dim3((s.M + 256 / (DD / 4) - 1) / (256 / (DD / 4)), BH), 256, 0, stream>>>(g, s.M)
        switch (s.d) {
            case 4: FLARE_EMF(4); break;
            case 8: FLARE_EMF(8); break;
            case 16: FLARE_EMF(16); break;
            case 32: FLARE_EMF(32); break;
            default: return FLARE_EUNSUPPORTED;
        }
#undef FLARE_EMF
        return check_launch();
    }
    switch (s.d) {
        case 4: encode_merge_kernel<4><<<blocks, 256, 0, stream>>>(m_part, l_part, o_part, z, lse_enc, BH, s.M, parts, s.dtype == FLARE_F32); break;
        case 8: encode_merge_kernel<8><<<blocks, 256, 0, stream>>>(m_part, l_part, o_part, z, lse_enc, BH, s.M, parts, s.dtype == FLARE_F32); break;
        case 16: encode_merge_kernel<16><<<blocks, 256, 0, stream>>>(m_part, l_part, o_part, z, lse_enc, BH, s.M, parts, s.dtype == FLARE_F32); break;
        case 32: encode_merge_kernel<32><<<blocks, 256, 0, stream>>>(m_part, l_part, o_part, z, lse_enc, BH, s.M, parts, s.dtype == FLARE_F32); break;
        default: return FLARE_EUNSUPPORTED;
    }
    return check_launch();
}

ValuPlan valu_plan(const flare_shape &s)
{
    ValuPlan p;
    const int BH = s.B * s.H;
    // chunks of at least 64 tokens: short sequences with few heads still spread over the chip; and of at
    // most 8192: a thread adds its chunk's terms one after the other in fp32, and the rounding of such a
    // sum grows with the square root of its length (the partial results are then combined by a tree)
    p.enc = plan_split(s.N, BH, 64, 2048);
    constexpr int kMaxChunk = 8192;
    if (p.enc.chunk_len > kMaxChunk) {
        p.enc.chunk_len = kMaxChunk;
        p.enc.chunks = (s.N + kMaxChunk - 1) / kMaxChunk;
    }
    if (s.dtype == FLARE_F32) p.enc = mfma32_split(s);
    p.bwd = p.enc;
    p.fwd_bytes = valu_fwd_layout(s, p.enc, nullptr, nullptr, nullptr, nullptr);
    return p;
}
// (apart from the plan, which every forward call makes two or three times over: the slots of dZ and dQ take the counts of four kernels)
size_t valu_bwd_bytes(const flare_shape &s) { return bwd_layout(s, valu_plan(s), nullptr, nullptr); }

int valu_encode(const flare_shape &s, const void *q, const void *k, const void *v, float *z, float *lse_enc,
                float scale, void *ws, hipStream_t stream)
{
    FLARE_DISPATCH(s, (encode_impl<T, D>(s, (const T *)q, (const T *)k, (const T *)v, z, lse_enc, scale, ws, stream)));
}
int valu_forward(const flare_shape &s, const void *q, const void *k, const void *v, void *y, float *z, float *lse_enc,
                 float *lse_dec, float scale, void *ws, hipStream_t stream)
{
    FLARE_DISPATCH(s, (forward_impl<T, D>(s, (const T *)q, (const T *)k, (const T *)v, (T *)y, z, lse_enc, lse_dec, scale,
                                          ws, stream)));
}
int valu_decode(const flare_shape &s, const void *q, const void *k, const float *z, void *y, float *lse_dec,
                float scale, hipStream_t stream)
{
    FLARE_DISPATCH(s, (decode_impl<T, D>(s, (const T *)q, (const T *)k, z, (T *)y, lse_dec, scale, stream)));
}
int valu_backward(const flare_shape &s, const void *q, const void *k, const void *v, const void *y,
                  const float *lse_dec, const void *dy, const float *z, const float *lse_enc, void *dq,
                  bool dq_cast, void *dk, void *dv, float scale, void *ws, hipStream_t stream)
{
    FLARE_DISPATCH(s, (backward_impl<T, D>(s, (const T *)q, (const T *)k, (const T *)v, (const T *)y, lse_dec,
                                           (const T *)dy, z, lse_enc, dq, dq_cast, (T *)dk, (T *)dv, scale, ws, stream)));
}

}  // namespace flare
