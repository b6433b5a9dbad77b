// Internal declarations shared by the translation units of libflare.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "flare.h"
#include "flare_profile.h"

namespace flare {

struct MergeZ;    // flare_merge.h
struct MergeDz;

// ---- kernel ids for the per-kernel timing hooks ------------------------------------------
enum KernelId {
    KID_ENCODE_PARTIAL = 0,
    KID_ENCODE_MERGE,
    KID_DECODE,
    KID_BWD_TOKEN_STATS,
    KID_BWD_PREP,
    KID_BWD_DZ_PARTIAL,
    KID_BWD_DZ_MERGE,
    KID_BWD_DQ_PARTIAL,
    KID_BWD_DQ_REDUCE,
    KID_BWD_DKDV,
    KID_DECODE_MERGE,
    KID_SPECTRAL_GRAM,
    KID_SPECTRAL_REDUCE,
    KID_SPECTRAL_EIGEN,
    KID_SPECTRAL_POST,
    KID_DECODE_PROJECT,
    KID_COUNT
};

// Brackets one launch with events when timing is on (see flare_profile_enable).
struct LaunchTimer {
    LaunchTimer(int kid, hipStream_t stream);
    ~LaunchTimer();
    int slot;
    hipStream_t stream;
};

// ---- how the token axis is split over workgroups -------------------------------------------
struct Split {
    int chunks;     // number of token chunks per (b,h)
    int chunk_len;  // tokens per chunk (the last chunk may be shorter, never empty)
};
Split plan_split(int N, int BH, int min_len, int target_blocks);

// ---- where a row of a token tensor (k, v, y, dy, dk, dv) lives --------------------------------
// Element (b, h, n, j) is at b*sb + h*sh + n*sn + j (in elements), for either layout of flare.h.
// sq: elements between the latent queries of consecutive heads (M*d, or 0 when all heads share one
// latent sequence): head h's queries start at q_lat + h*sq.
struct TokStride {
    long long sb, sh, sn, sq;
};
inline TokStride tok_stride(const flare_shape &s)
{
    const long long H = s.H, N = s.N, d = s.d;
    const long long sq = s.shared_latents ? 0 : (long long)s.M * d;
    if (s.layout == FLARE_BNHD) return TokStride{N * H * d, d, H * d, sq};
    return TokStride{H * N * d, N * d, d, sq};
}
__device__ __forceinline__ size_t tok_base(const TokStride &t, int bh, int H)
{
    return (size_t)(bh / H) * (size_t)t.sb + (size_t)(bh % H) * (size_t)t.sh;
}
// Offset of token n's row inside its (b,h) slice.  A full-rate 24-bit multiply: the entry points
// admit only shapes with N < 2^24 and N * sn < 2^32 (see check_shape).
__device__ __forceinline__ size_t tok_off(const TokStride &t, int n)
{
    return (size_t)__umul24((unsigned)n, (unsigned)t.sn);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// ---- fp32 vector-ALU path (any M, d in {4,8,16,32}, 16-bit storage), launch sequences of fp32 storage ---
struct ValuPlan {
    Split enc;          // split used by the encode partials
    Split bwd;          // split used by the dZ and dQ partials
    size_t fwd_bytes;   // workspace for encode
};
ValuPlan valu_plan(const flare_shape &s);
size_t valu_bwd_bytes(const flare_shape &s);   // workspace for backward

// Carves the encode workspace for sp.chunks partial slots per (b,h); returns its size in bytes.
// Any of the output pointers may be NULL (then ws is not touched).
size_t valu_fwd_layout(const flare_shape &s, const Split &sp, void *ws, float **m_part, float **l_part,
                       float **o_part);
// Fixed-order merge of `parts` partial slots per (b,h) into z and lse_enc (shared by both paths).
int launch_encode_merge(const flare_shape &s, const float *m_part, const float *l_part, const float *o_part,
                        float *z, float *lse_enc, int parts, hipStream_t stream);

int valu_encode(const flare_shape &s, const void *q, const void *k, const void *v, float *z,
                float *lse_enc, float scale, void *ws, hipStream_t stream);
int valu_forward(const flare_shape &s, const void *q, const void *k, const void *v, void *y, float *z, float *lse_enc,
                 float *lse_dec, float scale, void *ws, hipStream_t stream);
int valu_decode(const flare_shape &s, const void *q, const void *k, const float *z, void *y,
                float *lse_dec, float scale, hipStream_t stream);
// The whole backward; uses the matrix-core kernels where the shape allows.  y and lse_dec may be
// NULL (then the token statistics are recomputed).  dq is fp32, or of the storage type with dq_cast.
int valu_backward(const flare_shape &s, const void *q, const void *k, const void *v, const void *y,
                  const float *lse_dec, const void *dy, const float *z, const float *lse_enc, void *dq,
                  bool dq_cast, void *dk, void *dv, float scale, void *ws, hipStream_t stream);

// ---- matrix-core path of 16-bit storage (M <= 2048, N >= 16; mfma_supported) -----------------
struct MfmaPlan {
    Split enc;   // token chunks of the encode (one workgroup each)
    int parts;   // partial slots per (b,h) of the encode and dZ kernels: one per chunk
};
bool mfma_supported(const flare_shape &s);
MfmaPlan mfma_plan(const flare_shape &s);
size_t mfma_fwd_bytes(const flare_shape &s);
int mfma_encode(const flare_shape &s, const void *q, const void *k, const void *v, float *z,
                float *lse_enc, float scale, void *ws, hipStream_t stream);
// encode and decode; where the encode's slots are few the decode merges them itself
int mfma_forward(const flare_shape &s, const void *q, const void *k, const void *v, void *y, float *z, float *lse_enc,
                 float *lse_dec, float scale, void *ws, hipStream_t stream);
// The encode's partial slots only; *g says where they are, for a consumer to merge.
int mfma_encode_partial(const flare_shape &s, const void *q, const void *k, const void *v, float *z, float *lse_enc,
                        float scale, void *ws, MergeZ *g, hipStream_t stream);
// Shapes with M > 256 run the token-major kernels once per chunk of at most 256 latents.  The decode then needs
// mfma_tok_run_bytes(s) of scratch, the token statistics mfma_tok_stats_bytes(s) (`ws`; unused and may be NULL
// otherwise), the dK/dV step mfma_dkdv_acc_bytes(s) for its fp32 sums.
size_t mfma_tok_run_bytes(const flare_shape &s);
size_t mfma_tok_stats_bytes(const flare_shape &s);
size_t mfma_dkdv_acc_bytes(const flare_shape &s);
int mfma_lat_step(const flare_shape &s);   // latents per chunk
int mfma_decode(const flare_shape &s, const void *q, const void *k, const float *z, void *y,
                float *lse_dec, float scale, void *ws, hipStream_t stream);
// decode fused with the output projection (flare_mfma_proj.hip); y and lse_dec may be NULL
bool mfma_project_supported(const flare_shape &s);
int mfma_decode_project(const flare_shape &s, const void *q, const void *k, const float *z, const void *w_out,
                        const float *bias, void *out, void *y, float *lse_dec, float scale, hipStream_t stream);
int mfma_token_stats(const flare_shape &s, const void *q, const void *k, const float *z, const void *dy,
                     float *lse_dec2, float *delta, float scale, void *ws, hipStream_t stream);
// In the backward launchers below the per-token decode statistic is read as
// ld_mul * lse_dec2[n]: pass the workspace array with ld_mul = 1, or the forward's natural-log
// lse_dec with ld_mul = log2(e).
int mfma_dkdv(const flare_shape &s, const void *q, const void *k, const void *v, const void *dy, const float *z,
              const float *lse_enc, const float *lse_dec2, const float *delta, float ld_mul, void *dk, void *dv,
              float *acc32, float *dq_part, int m0, float scale, const MergeDz &g, hipStream_t stream);
int mfma_dkdv_blocks(const flare_shape &s);
bool mfma_dq_fused(const flare_shape &s);
int mfma_dq_parts(const flare_shape &s);
int mfma_dq_partial(const flare_shape &s, const void *q, const void *k, const void *v, const void *dy,
                    const float *z, const float *lse_enc, const float *dz, const float *eps,
                    const float *lse_dec2, const float *delta, float ld_mul, const int *plan, float *dq_part,
                    float scale, hipStream_t stream);
// May the dK/dV kernel merge the dZ slots itself?
bool mfma_dz_inline(const flare_shape &s);
// y and delta_out may be NULL; when given, delta_out[b][h][n] = <dY_n, Y_n> is written as a by-product.
int mfma_dz_partial(const flare_shape &s, const void *q, const void *k, const void *dy, const float *lse_dec2,
                    float ld_mul, const void *y, float *delta_out, float *ld_range, float *dz_part, float scale,
                    hipStream_t stream);
// ---- fp32 storage on the matrix cores (flare_mfma_f32.hip) ------------------------------------
// Partial slots per (b,h) of the latent-major kernels (encode, dZ, dQ) = chunks of this split.
Split mfma32_split(const flare_shape &s);
int mfma32_encode(const flare_shape &s, const float *q, const float *k, const float *v, float *m_part, float *l_part,
                  float *o_part, float scale, hipStream_t stream);
int mfma32_decode(const flare_shape &s, const float *q, const float *k, const float *z, float *y, float *lse_dec,
                  float scale, const MergeZ &g, hipStream_t stream);
int mfma32_token_stats(const flare_shape &s, const float *q, const float *k, const float *z, const float *dy,
                       float *lse_dec2, float *delta, float scale, hipStream_t stream);
// y, delta_out, ld_mul, ld_range, plan: as for the 16-bit launchers above
int mfma32_dz_partial(const flare_shape &s, const float *q, const float *k, const float *dy, const float *lse_dec,
                      float ld_mul, const float *y, float *delta_out, float *ld_range, float *dz_part, float scale,
                      hipStream_t stream);
int mfma32_dq_partial(const flare_shape &s, const float *q, const float *k, const float *v, const float *dy,
                      const float *z, const float *lse_enc, const float *dz, const float *eps, const float *lse_dec,
                      const float *delta, float ld_mul, const int *plan, float *dq_part, float scale, hipStream_t stream);
int mfma32_dkdv(const flare_shape &s, const float *q, const float *k, const float *v, const float *dy, const float *z,
                const float *lse_enc, const float *lse_dec, const float *delta, float ld_mul, float *dk, float *dv,
                float *dq_part, float scale, const MergeDz &g, hipStream_t stream);
// Does the dK/dV kernel also form the dQ partials (dq_part != NULL above)?  Its slots per (b,h) then (0: it does not).
bool mfma32_dq_fused(const flare_shape &s);
int mfma32_dq_blocks(const flare_shape &s);
bool mfma32_inline(const flare_shape &s);   // do the decode and dK/dV kernels merge the slots?

// ---- spectral analysis (Appendix C.1, Algorithm 1) ---------------------------------------------
bool mfma_gram_supported(const flare_shape &s);
int mfma_gram_partial(const flare_shape &s, const Split &sp, const void *q, const void *k, const float *lse_enc,
                      const float *lse_dec, float *g_part, float scale, hipStream_t stream);
size_t spectral_bytes(const flare_shape &s);
int spectral_run(const flare_shape &s, const void *q, const void *k, const float *lse_enc, const float *lse_dec,
                 float scale, int first, float *evals, float *zvec, float *gram, void *ws, hipStream_t stream);

}  // namespace flare
