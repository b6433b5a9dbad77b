// Matrix-core kernels of the second backward pass: dQ, dK, dV (one kernel; two with FLARE_VARIANT_SEPARATE_DQ),
// the per-(b,h) choice between the one- and two-exponential variants, and the fp32 sums of latent chunks.
// Operand layouts, helpers and the tile geometry are in flare_mfma_common.h.
#include "flare_mfma_common.h"

namespace flare {
namespace {

// ============================================================================================
// Backward, dQ partials (latent-major, same wave geometry as the encode), where the dK/dV kernel is asked to leave them
// out (FLARE_VARIANT_SEPARATE_DQ).  For its NB latent tiles
// a wave keeps, as B operands (column = latent, contraction over d): q' hi and lo, dZ (bf16-exact: it is
// rounded where it is merged, before eps is formed) and Z in bf16 (hi and, at d = 16, lo).  Per 32-token tile it streams K, V and dY as A operands
// (row = token) and forms, all on the matrix cores,
//     S2 - lse_enc2[m]   (one more k-step: -lse_enc2 as a hi+lo pair in slots 0,1, against 1,1)
//     S2 - lse_dec2[n]   (likewise -lse_dec2 in slots 2,3 of the token-side operand)
//     a[n][m] = <V_n, dZ_m> - eps[m]      (-eps rides in one more, otherwise empty, k-step)
//     c[n][m] = <dY_n, Z_m> - delta[n]    (-delta likewise)
// then dS^T = 2^(..) a + 2^(..) c in fp32, rounds it to bf16 and accumulates
//     dQ^T[dd][m] += K^T[dd][n] dS^T[n][m]
// with K^T read back from a wave-private, double-buffered LDS tile.  Masked tokens have both
// exponents at -inf, so their dS is exactly zero.
//
// ONE = true is the variant with one exponential per score, P~ = 2^S2 without a normaliser:
//     P = P~ e[m],  R = P~ w[n],   e[m] = 2^-lse_enc2[m],  w[n] = 2^-lse_dec2[n],
// so dS^T = P~ (e[m] (a - eps) + w[n] (c - delta)).  e[m] arrives folded into dZ and eps (the kernel that merges
// the dZ partials scales dZ before it rounds it and forms eps), so the a chain needs nothing new and the score
// products need no correction k-step; w[n] is a per-row factor that goes from the token's lane to the rows of
// the accumulator layout through 128 bytes of LDS (and multiplies delta in the correction k-step).  It is exact
// as long as both log-sum-exps stay within +-60, which bwd_one_exp_ok checks per (b,h) (plan[bh] = 1);
// otherwise the ONE = false variant runs.  Each variant returns at once when the plan names the other.
// ============================================================================================
template <int DR, int NB, int MINB, bool ONE, bool F>
__device__ __forceinline__ void dq_body(
    const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ dy, const float *__restrict__ z, const float *__restrict__ lse_enc,
    const float *__restrict__ dz, const float *__restrict__ eps, const float *__restrict__ lse_dec2,
    const float *__restrict__ delta, float ld_mul, float *__restrict__ dq_part,
    TokStride ts, int H, int N, int M, int chunk_len, int parts, int G, int TG, float c2)
{
    // dz, eps: the rows of this (b,h)
    constexpr int D = padded_dim(DR);
    constexpr int KS = D / 16;
    // Row blocks of the dQ accumulation.  d <= 16: one 32x32 product per 16 columns (rows 16-31 of the K^T
    // operand are zero).  d = 32: the 32 columns fill the 32 rows of ONE product (WIDE).
    constexpr bool WIDE = (D == 32);
    constexpr int HV = WIDE ? 1 : D / 16;
    constexpr int QUARTS = WIDE ? 4 : 2;        // 4-column pieces per lane and accumulator: columns 8 q + 4 hh (+ 16 hv)
    constexpr int ROWS = D + 1;                 // K^T rows, then a row of zeros
    // d <= 8: the upper half of the padded contraction carries what otherwise needs products of its own:
    // q' lo and Z lo (K and dY rows repeated in both lane halves) and -eps (against ones in the V operand).
    constexpr bool PACK = pack_dim(DR);
    // d = 32: the key tile goes to LDS as loaded, row = token (kKwStride uint16 a row: 80 B, two 16-byte stores per
    // lane), and the transposing read forms the K^T operand; d <= 16: transposed on the way in, two bytes a store.
    constexpr int kKwStride = 40;
    constexpr int BUF = WIDE ? 32 * kKwStride : ROWS * kVtStride;
    __shared__ __attribute__((aligned(16))) uint16_t kt_all[4][2 * BUF];
    __shared__ __attribute__((aligned(16))) float wl_all[ONE ? 4 : 1][2][32];   // w[n] of a token tile

    const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // known to be wave-uniform: scalar unit
    const int g = wave % G, tg = wave / G;
    const GridPos gp = grid_pos(ts, H, DR * 2);
    const int bh = gp.y, h = bh % H, chunk = gp.x;
    const bool lower = hh == 0;
    uint16_t *lds = kt_all[wave];
    float (*wl)[32] = wl_all[ONE ? wave : 0];
    constexpr float kap = 0.f;                  // w[n] = 2^(kap - lse_dec2[n])
    if (!WIDE && lane < kVtStride) {
        lds[D * kVtStride + lane] = 0;
        lds[BUF + D * kVtStride + lane] = 0;
        if constexpr (PACK) {   // K^T rows 8-15 are never written: zero, so that the unused output rows stay finite
#pragma unroll
            for (int r = 8; r < 16; ++r) {
                lds[r * kVtStride + lane] = 0;
                lds[BUF + r * kVtStride + lane] = 0;
            }
        }
    }

    // ---- per-latent operands ----
    const int lat0 = 32 * NB * (G * (int)blockIdx.z + g);   // a workgroup owns NB*G tiles of latents
    constexpr bool LO2 = (D == 16);             // carry the lo term of Z as well (dZ arrives bf16-exact)
    bf16x8 qh[NB][KS], ql[NB][KS], q_aug[NB], dzb[NB][KS], zb[NB][KS], zl[NB][KS], dz_aug[NB];
    bf16x8 u_aug[ONE ? NB : 1];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        // padding latents (at or beyond M): every operand zero, loads clamped to the last real latent
        const bool real = lat0 + 32 * b + l32 < M;
        const int m = min(lat0 + 32 * b + l32, M - 1);
        load_q_operand<DR, true, F, PACK>(q + (size_t)h * ts.sq + (size_t)m * DR, hh, c2, false, qh[b], ql[b]);
        if (!real) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { qh[b][ks] = zero_operand(); ql[b][ks] = zero_operand(); }
        }
        const float le2 = real ? lse_enc[(size_t)bh * M + m] * kLog2e : 0.f;
        const float um = 1.f;                       // (a per-latent factor of the c chain: none in either variant)
        if constexpr (ONE) {
            const uint32_t us = split_bf16_pair(um);          // slots 0,1,2 := u hi, u hi, u lo
            u32x4 wu;
            wu[0] = lower ? ((us & 0xffffu) | (us << 16)) : 0u;
            wu[1] = lower ? (us >> 16) : 0u;
            // slots 4,5 := -eps (hi + lo): with one exponential the a chain's correction rides in the same
            // product as the c chain's (against ones in the token operand), see the tile loop
            wu[2] = (!PACK && lower) ? split_bf16_pair(real ? -eps[m] : 0.f) : 0u;
            wu[3] = 0u;
            u_aug[b] = as_bf16x8(wu);
        }
        u32x4 wq;
        wq[0] = lower ? split_pair<F>(-le2) : 0u;       // slots 0,1 := -lse_enc2 (hi + lo)
        wq[1] = lower ? kOnePair<F> : 0u;               // slots 2,3 := 1
        wq[2] = 0u; wq[3] = 0u;
        q_aug[b] = as_bf16x8(wq);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            float zr[8], dr[8];
            row8_f32<DR>(z + ((size_t)bh * M + m) * DR, PACK ? 0 : (D / 2) * hh + 8 * s, zr);
            row8_f32<DR>(dz + (size_t)m * DR, (D / 2) * hh + 8 * s, dr);
            if (!real) {
#pragma unroll
                for (int i = 0; i < 8; ++i) { zr[i] = 0.f; dr[i] = 0.f; }
            }
            u32x4 wz, wd, wzl;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float za = zr[2 * i] * um, zc = zr[2 * i + 1] * um;
                const uint32_t z0 = rne_bf16(za), z1 = rne_bf16(zc);
                const uint32_t d0 = rne_bf16(dr[2 * i]), d1 = rne_bf16(dr[2 * i + 1]);
                wz[i] = z0 | (z1 << 16);
                wd[i] = d0 | (d1 << 16);
                wzl[i] = rne_bf16(za - __uint_as_float(z0 << 16)) |
                         (rne_bf16(zc - __uint_as_float(z1 << 16)) << 16);
            }
            zb[b][s] = as_bf16x8((PACK && !lower) ? wzl : wz);
            dzb[b][s] = as_bf16x8(wd);
            zl[b][s] = as_bf16x8(wzl);
        }
        u32x4 we;
        we[0] = (lower != PACK) ? split_bf16_pair(real ? -eps[m] : 0.f) : 0u;
        we[1] = 0u; we[2] = 0u; we[3] = 0u;
        dz_aug[b] = as_bf16x8(we);
        if constexpr (PACK) {   // slots 8,9 of the dZ operand := -eps (the rest of its upper half is zero)
            u32x4 wd = __builtin_bit_cast(u32x4, dzb[b][0]);
            if (!lower) wd[0] = we[0];
            dzb[b][0] = as_bf16x8(wd);
        }
    }
    u32x4 w11;
    w11[0] = lower ? 0x3f803f80u : 0u;
    w11[1] = 0u; w11[2] = 0u; w11[3] = 0u;
    const bf16x8 ones_aug = as_bf16x8(w11);      // slots 0,1 = 1 in the lower lane half, else 0
    w11[0] = lower ? kOnePair<F> : 0u;
    const bf16x8 ones_s = as_bf16x8(w11);        // the same in the type of the score products
    auto to_bf16 = [](bf16x8 x) { return as_bf16x8(to_bf16_row<F>(__builtin_bit_cast(u32x4, x))); };
    // V rows as the operand of the a product; PACK: slots 8,9 := 1 (the upper lane half loaded zeros)
    auto v_operand = [&](bf16x8 x) {
        u32x4 w = to_bf16_row<F>(__builtin_bit_cast(u32x4, x));
        if (PACK && !lower) w[0] = 0x3f803f80u;
        return as_bf16x8(w);
    };

    const bf16_t *kb = k + tok_base(ts, bh, H);
    const bf16_t *vb = v + tok_base(ts, bh, H);
    const bf16_t *gb = dy + tok_base(ts, bh, H);
    const float *lb = lse_dec2 + (size_t)bh * N;
    const float *db = delta + (size_t)bh * N;
    const int n0 = chunk * chunk_len;
    const int n1 = min(N, n0 + chunk_len);
    const int tiles = (n1 - n0 + 31) / 32;
    const int cnt = (tiles > tg) ? (tiles - tg + TG - 1) / TG : 0;

    f32x16 acc[NB][HV];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int hv = 0; hv < HV; ++hv) acc[b][hv] = splat16(0.f);

    int krow[HV];
#pragma unroll
    for (int hv = 0; hv < HV; ++hv) krow[hv] = WIDE ? l32 : ((l32 < 16) ? 16 * hv + l32 : D);

    auto tile_tok0 = [&](int j) { return n0 + 32 * (tg + min(j, cnt - 1) * TG); };
    // A operand: row = token.  rep (PACK only): both lane halves get elements 0-7 of the row.
    auto load_rows = [&](const bf16_t *base, int j, bf16x8 (&t)[KS], bool rep) {
        const int n = min(tile_tok0(j) + l32, N - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s)
            t[s] = as_bf16x8(row8_bf16<DR>(base + tok_off(ts, n), (PACK && rep) ? 0 : (D / 2) * hh + 8 * s));
    };
    auto write_kt = [&](const bf16x8 (&t)[KS], uint16_t *buf) {   // transposed: row = d-index, column = token
        if (PACK && !lower) return;   // the upper lane half holds a copy of the same elements
        if constexpr (WIDE) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                *reinterpret_cast<u32x4 *>(buf + l32 * kKwStride + (D / 2) * hh + 8 * s) =
                    to_bf16_row<F>(__builtin_bit_cast(u32x4, t[s]));
            return;
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const u32x4 w = to_bf16_row<F>(__builtin_bit_cast(u32x4, t[s]));   // K as a value: bf16
            const int d0 = (D / 2) * hh + 8 * s;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                buf[(d0 + 2 * e) * kVtStride + l32] = (uint16_t)(w[e] & 0xffffu);
                buf[(d0 + 2 * e + 1) * kVtStride + l32] = (uint16_t)(w[e] >> 16);
            }
        }
    };
    auto read_kT = [&](const uint16_t *buf, bf16x8 (&kT)[HV][2]) {
#pragma unroll
        for (int hv = 0; hv < HV; ++hv)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                if constexpr (WIDE) {
                    // lanes 16 i .. 16 i + 15 hand in four rows (tokens) of 16 columns (d-indices 16 (i & 1) ..) and
                    // lane c of them receives column c of the four: tokens 16 s2 + 4 hh + 0..3, then + 8..11
                    const int c16 = lane & 15;
                    const uint16_t *src =
                        buf + (16 * s2 + 4 * hh + (c16 >> 2)) * kKwStride + 16 * (l32 >> 4) + 4 * (c16 & 3);
                    const u32x2 a = lds_read_tr16(src), b = lds_read_tr16(src + 8 * kKwStride);
                    kT[hv][s2] = as_bf16x8(u32x4{a[0], a[1], b[0], b[1]});
                    continue;
                }
                const uint16_t *row = buf + krow[hv] * kVtStride + 16 * s2 + 4 * hh;
                const u32x2 a = *reinterpret_cast<const u32x2 *>(row);
                const u32x2 b = *reinterpret_cast<const u32x2 *>(row + 8);
                u32x4 w;
                w[0] = a[0]; w[1] = a[1]; w[2] = b[0]; w[3] = b[1];
                kT[hv][s2] = as_bf16x8(w);
            }
    };

    // w[n] of a tile: written by the token's lane, read back as the 16 rows of this lane's registers
    auto read_w = [&](const float *buf, float (&wr)[16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 t = *reinterpret_cast<const float4 *>(buf + 8 * i + 4 * hh);
            wr[4 * i] = t.x; wr[4 * i + 1] = t.y; wr[4 * i + 2] = t.z; wr[4 * i + 3] = t.w;
        }
    };

    if (cnt > 0) {
        // The rows of a token tile (keys, values, dY, as loaded) and its two statistics are requested as soon as
        // the tile three places earlier is done with its registers: a tile of this kernel is short (one or two
        // latent tiles), and a request has to be older than the memory latency when its rows are needed (the keys
        // two tiles later, the rest three).  Three sets of registers take turns as current tile, next tile and in
        // flight, so that no register of a load in flight is ever copied.
        struct Rows {
            bf16x8 k[KS], v[KS], g[KS];
            float l, d;   // lse_dec2 as stored, delta
        };
        auto request = [&](int j, Rows &r) {
            load_rows(kb, j, r.k, true);
            load_rows(vb, j, r.v, false);
            load_rows(gb, j, r.g, true);
            const int n = min(tile_tok0(j) + l32, N - 1);
            r.l = lb[n];
            r.d = db[n];
        };
        Rows ra, rb, rc;
        bf16x8 kT[HV][2];
        float wrow[ONE ? 16 : 1];
        request(0, ra);
        request(1, rb);
        request(2, rc);
        compiler_fence();
        write_kt(ra.k, lds);
        if constexpr (ONE) wl[0][l32] = fast_exp2(kap - ra.l * ld_mul);
        compiler_fence();
        read_kT(lds, kT);
        if constexpr (ONE) read_w(wl[0], wrow);

        // tile j: cur holds its rows (and receives those of tile j+3 at the end), nxt those of tile j+1
        auto tile = [&](int j, Rows &cur, const Rows &nxt) {
            const int tok0 = tile_tok0(j);
            uint16_t *buf_next = lds + ((j + 1) & 1) * BUF;
            const float nld = -cur.l * ld_mul, dl = cur.d;
            bf16x8 vt[KS], gt[KS];   // V and dY meet bf16 operands
#pragma unroll
            for (int s = 0; s < KS; ++s) { vt[s] = v_operand(cur.v[s]); gt[s] = to_bf16(cur.g[s]); }

            // token-side operands of the correction k-steps (zero outside the named slots)
            u32x4 wb;
            wb[0] = 0u; wb[2] = 0u; wb[3] = 0u;
            wb[1] = lower ? split_pair<F>(nld) : 0u;             // slots 2,3 := -lse_dec2[n]
            const bf16x8 kt_a = ones_s, kt_b = as_bf16x8(wb);    // slots 0,1 := 1 picks -lse_enc2
            // One exponential (d >= 16): dS = P (a + w c) and w[n] is this lane's token's, so ONE product serves
            // both corrections: slots 0,1,2 = -w delta (hi, lo, hi) meet u (hi, hi, lo) and slots 4,5 = 1 pick
            // -eps; the a chain starts from it and the c chain from zero.
            constexpr bool MERGED = ONE && !PACK;
            u32x4 wg;
            const uint32_t ds_ = split_bf16_pair(MERGED ? -dl * fast_exp2(kap + nld) : -dl);
            wg[0] = lower ? ds_ : 0u;
            wg[1] = (ONE && lower) ? (ds_ & 0xffffu) : 0u;       // ONE: slots 0,1,2 := -delta hi, lo, hi
            wg[2] = (MERGED && lower) ? 0x3f803f80u : 0u;
            wg[3] = 0u;
            const bf16x8 g_aug = as_bf16x8(wg);

            const int rem = n1 - tok0 - 4 * hh;
            const bool partial = tok0 + 32 > n1;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                f32x16 x = splat16(0.f);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) x = mfma_s<F>(cur.k[ks], qh[b][ks], x);
                if constexpr (!PACK) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) x = mfma_s<F>(cur.k[ks], ql[b][ks], x);
                }
                f32x16 s1 = x;                  // one exponential: the scores as they are
                if constexpr (!ONE) s1 = mfma_s<F>(kt_a, q_aug[b], x);
                f32x16 s2 = s1;
                if constexpr (!ONE) s2 = mfma_s<F>(kt_b, q_aug[b], x);
                f32x16 av = splat16(0.f), cv = splat16(0.f);
                if constexpr (MERGED) {
                    av = mfma(g_aug, u_aug[ONE ? b : 0], av);
                } else {
                    if constexpr (!PACK) av = mfma(ones_aug, dz_aug[b], av);
                    cv = mfma(g_aug, ONE ? u_aug[ONE ? b : 0] : ones_aug, cv);
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    av = mfma(vt[ks], dzb[b][ks], av);
                    cv = mfma(gt[ks], zb[b][ks], cv);
                    if constexpr (LO2 && !PACK) cv = mfma(gt[ks], zl[b][ks], cv);
                }
                if (partial) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r / 4) + (r % 4) >= rem) { s1[r] = -INFINITY; s2[r] = -INFINITY; }
                }
                f32x16 ds;
                if constexpr (ONE) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) ds[i] = fast_exp2(s1[i]) * fmaf(cv[i], wrow[i], av[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) ds[i] = fmaf(fast_exp2(s2[i]), cv[i], fast_exp2(s1[i]) * av[i]);
                }
                u32x4 w0, w1;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    w0[i] = cvt_pk_bf16(ds[2 * i], ds[2 * i + 1]);
                    w1[i] = cvt_pk_bf16(ds[8 + 2 * i], ds[8 + 2 * i + 1]);
                }
#pragma unroll
                for (int hv = 0; hv < HV; ++hv) {
                    acc[b][hv] = mfma(kT[hv][0], as_bf16x8(w0), acc[b][hv]);
                    acc[b][hv] = mfma(kT[hv][1], as_bf16x8(w1), acc[b][hv]);
                }
            }
            // The next tile's K^T and w go through LDS here, at the end of the tile: its rows were requested two
            // tiles ago, and what is read back is first needed by the last products of the next tile.
            compiler_fence();
            write_kt(nxt.k, buf_next);
            if constexpr (ONE) wl[(j + 1) & 1][l32] = fast_exp2(kap - nxt.l * ld_mul);
            compiler_fence();
            request(j + 3, cur);
            read_kT(buf_next, kT);
            if constexpr (ONE) read_w(wl[(j + 1) & 1], wrow);
            sched_fence();   // consecutive tiles are not interleaved (their temporaries would not fit the registers)
        };
        int j = 0;
        for (; j + 3 <= cnt; j += 3) {
            tile(j, ra, rb);
            tile(j + 1, rb, rc);
            tile(j + 2, rc, ra);
        }
        if (j < cnt) {
            tile(j, ra, rb);
            if (j + 1 < cnt) tile(j + 1, rb, rc);
        }
    }

    const size_t part = (size_t)bh * parts + (size_t)chunk * TG + tg;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (lat0 + 32 * b + l32 >= M) continue;
        const size_t slot = part * M + lat0 + 32 * b + l32;
#pragma unroll
        for (int hv = 0; hv < HV; ++hv)
#pragma unroll
            for (int qd = 0; qd < QUARTS; ++qd) {
                const int o = 16 * hv + 8 * qd + 4 * hh;
                if (o >= DR) continue;
                *reinterpret_cast<float4 *>(dq_part + slot * DR + o) = make_float4(
                    acc[b][hv][4 * qd], acc[b][hv][4 * qd + 1], acc[b][hv][4 * qd + 2], acc[b][hv][4 * qd + 3]);
            }
    }
}

// Both variants in one launch: each workgroup takes the one that the plan names for its (b,h) (a second launch whose
// workgroups all leave at once would still cost 4-6 us).  The two bodies share the kernel's registers; their LDS adds up.
template <int DR, int NB, int MINB, bool F>
__global__ __launch_bounds__(256, MINB) void bwd_dq_mfma_kernel(
    const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ dy, const float *__restrict__ z, const float *__restrict__ lse_enc,
    const float *__restrict__ dz, const float *__restrict__ eps, const float *__restrict__ lse_dec2,
    const float *__restrict__ delta, float ld_mul, const int *__restrict__ plan, float *__restrict__ dq_part,
    TokStride ts, int H, int N, int M, int chunk_len, int parts, int G, int TG, float c2)
{
    const int bh = grid_pos(ts, H, DR * 2).y;
    const float *dz_bh = dz + (size_t)bh * M * DR, *eps_bh = eps + (size_t)bh * M;
    if (plan[bh] != 0)
        dq_body<DR, NB, MINB, true, F>(q, k, v, dy, z, lse_enc, dz_bh, eps_bh, lse_dec2, delta, ld_mul, dq_part, ts, H, N, M,
                                       chunk_len, parts, G, TG, c2);
    else
        dq_body<DR, NB, MINB, false, F>(q, k, v, dy, z, lse_enc, dz_bh, eps_bh, lse_dec2, delta, ld_mul, dq_part, ts, H, N, M,
                                        chunk_len, parts, G, TG, c2);
}

// ============================================================================================
// Backward, dK and dV (token-major, like the decode: one wave owns 32 tokens at a time and walks
// over all latent tiles).  Everything that depends on the latents only is prepared once per
// workgroup as MFMA-ready operand images in LDS (one (b,h) per workgroup, 8 waves share it):
//   A-type images (row = latent, contraction over d): q' hi, q' lo, dZ hi (and lo), Z hi (and
//     lo), and a correction operand (slots 0,1 = -lse_enc2 as a hi+lo pair, slots 2,3 = 1,1; slots
//     8,9 = -eps as a hi+lo pair; slots 10,11 = 1,1 or, with one exponential, slots 4-6 = u: they
//     pick -delta[n] out of the token-side operand of the c chain's correction k-step);
//   row images (row = output column, contraction over the 32 latents in accumulator order):
//     RW1 = [dZ^T ; 0]   and   RW2 = [q^T ; 0]   (d = 32: all 32 rows are columns of dZ and q).
// Per token tile and latent tile:  P = 2^(S2 - lse_enc2[m]), R = 2^(S2 - lse_dec2[n]),
//   a = <dZ_m, V_n> - eps[m],  c = <Z_m, dY_n> - delta[n],  dS = P a + R c  (fp32), then
//   acc1 += RW1 . P   (rows 0-15: dV^T)
//   acc2 += RW2 . dS  (rows 0-15: (sum_m dS q_m)^T)
// and at the end  dV = acc1[0:16],  dK = scale * acc2[0:16].
// (eps is subtracted inside the a chain, by one more product, so that a - eps = <dZ_m, V_n - Z_m>
// cancels before dS is rounded: where a latent attends sharply to tokens of similar values the two
// terms agree to several digits, and carrying -eps q separately through bf16 roundings lost them.)
// No lo terms of dZ and Z for dK and dV: dZ arrives bf16-exact, and the rounding of Z_m is one error per
// latent, which the sums of dK_n and dV_n over the latents average out (measured: dK error up by
// 5-10 %, time down by 9 %) -- unlike in dQ, whose sums run over the tokens of one latent and add that
// error up coherently (the DQ variant below therefore carries the lo term of Z at d <= 8, and at d = 16 where the
// shape calls for it: ZL).
// ONE: one exponential per score, as in the dQ kernel: R = P u[m] w[n]; u is folded into the Z images
// (and into slots 4-6 of the correction image, against -delta in the token operand), w[n] is a
// per-lane scalar here, and dS' = P (a + w c).  Runs only where plan[bh] = 1.
// ============================================================================================
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kDsStride = 36;   // uint16 per row of the dS tile [token][latent] (72 B: conflict-free 8-byte stores)
// uint16 per row of the key tile [token][d] of the fused dQ product (rows as loaded; d = 32: 80 B, two 16-byte stores)
constexpr int kt_stride(int d) { return d == 32 ? 40 : 16; }
// uint16 per wave: dS tile (at least as long as an accumulator where two waves share a token tile, which they exchange
// there), then the key tile
constexpr bool dkdv_pair(int d, int mt) { return d == 32 && mt > 4; }
constexpr int ds_tile_lds(int d, int mt) { return dkdv_pair(d, mt) ? 64 * 16 * 2 : 32 * kDsStride; }
constexpr int fused_wave_lds(int d, int mt) { return ds_tile_lds(d, mt) + 32 * kt_stride(d); }

// operand images per latent tile: A-type ones (the last: corrections), then row images (RW1, RW2) x 2 k-steps
constexpr int dkdv_a_images(int dr, bool dq, bool zl) { return (dq && !pack_dim(dr) && zl ? 5 : 4) * (padded_dim(dr) / 16) + 1; }
constexpr int dkdv_images(int dr, bool dq, bool zl) { return dkdv_a_images(dr, dq, zl) + 4; }

constexpr int WV = 8;           // waves per workgroup (one workgroup per CU)

// The latents' rows of z and q and their lse_enc in LDS while the operand images are built from them: in the part that the
// waves' dS and key tiles take afterwards.  (Each image reading its elements from global memory waited for them seven
// times over, at 128 latents and d = 32.)
template <int DR>
struct LatentStage {
    float *z, *lse;
    bf16_t *q;
    __device__ __forceinline__ LatentStage(void *at, int M)
    {
        z = static_cast<float *>(at);
        q = reinterpret_cast<bf16_t *>(z + M * DR);
        lse = reinterpret_cast<float *>(q + M * DR);
    }
    static constexpr int kBytes = DR * 6 + 4;   // per latent
};
// (requested and put away apart, so that what is merged meanwhile waits for memory at the same time)
template <int DR, int MT>
struct LatentPieces {
    static_assert(LatentStage<DR>::kBytes * 32 * MT <= WV * fused_wave_lds(padded_dim(DR), MT) * 2, "as long as the waves' tiles");
    static constexpr int NT = 64 * WV, P = (32 * MT * DR / 4 + NT - 1) / NT;   // pieces of four columns a thread
    float4 z[P];
    u32x2 q[P];
    float lse;
    __device__ __forceinline__ void request(const bf16_t *qr, const float *zr, const float *lr, int M)
    {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int at = min((int)threadIdx.x + i * NT, M * DR / 4 - 1);
            z[i] = reinterpret_cast<const float4 *>(zr)[at];
            q[i] = reinterpret_cast<const u32x2 *>(qr)[at];
        }
        lse = lr[min((int)threadIdx.x, M - 1)];
    }
    __device__ __forceinline__ void put(void *where, int M) const
    {
        const LatentStage<DR> st(where, M);
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int at = (int)threadIdx.x + i * NT;
            if (at >= M * DR / 4) continue;
            reinterpret_cast<float4 *>(st.z)[at] = z[i];
            reinterpret_cast<u32x2 *>(st.q)[at] = q[i];
        }
        if ((int)threadIdx.x < M) st.lse[threadIdx.x] = lse;
    }
};

template <int DR, int MT, bool DQ, bool ONE, bool F, bool ZL = false>
__device__ __forceinline__ void dkdv_body(
    const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ dy, const float *__restrict__ z, const float *__restrict__ lse_enc,
    const float *__restrict__ dz, const float *__restrict__ eps, const float *__restrict__ lse_dec2,
    const float *__restrict__ delta, float ld_mul, bf16_t *__restrict__ dk,
    bf16_t *__restrict__ dv, float *__restrict__ acc32, float *__restrict__ dq_part, TokStride ts, int H, int N,
    int Mtot, int m0, int mend, float c2, float scale)
{
    // DQ: the kernel also forms the dQ partials, so that the scores, a, c and dS of a tile
    // pair are computed once for all three gradients.  dS of a tile reaches the dQ product transposed
    // (contraction over the tokens) through a wave-private LDS tile, and that product is
    //     dQ^T[dd][m] += K^T[dd][n] dS^T[n][m]     with v_mfma_f32_16x16x32_bf16
    // (16 output rows = d, two such products at d = 32: no wasted rows, four accumulator registers per 16 latents), so a
    // wave keeps dQ of all 32*MT latents in 8*MT registers (d = 32: 16*MT).  At the end the eight waves add their partials in a
    // fixed order through LDS and the workgroup writes slot x (its grid position) of dq_part
    // ([(b*h) * gridDim.x + x][Mtot][d], summed and scaled by dq_reduce_kernel).  The c chain
    // then carries the lo term of Z at d <= 8 (ZPACK below) and, with ZL, at d = 16 (dQ sums dS over the tokens of
    // one latent and adds up its rounding coherently, see the dQ kernel).
    // The kernel works on the latents m0 .. mend (at most 32 * MT) of the head's Mtot.  With acc32 given (more than one
    // latent chunk) it adds its dV and dK rows in fp32 to acc32[0][b*h][n][DR] and acc32[1][...] (the
    // chunk with m0 = 0 stores instead); the last chunk adds what is there to its own rows and rounds the
    // sums to dk and dv.  The chunks run as launches in a row on one stream, so the order of the sum is fixed.
    constexpr int D = padded_dim(DR);
    constexpr int KS = D / 16;
    // Row blocks of the two accumulations.  d <= 16: one 32x32 product per 16 columns (rows 16-31 of its
    // operand image are zero).  d = 32: the 32 columns fill the 32 rows of ONE product (WIDE), half the
    // matrix instructions of two half-empty ones.
    constexpr bool WIDE = (D == 32);
    constexpr int HV = WIDE ? 1 : D / 16;
    constexpr int QUARTS = WIDE ? 4 : 2;        // 4-column pieces per lane and accumulator: columns 8 q + 4 hh (+ 16 hv)
    // PAIR (d = 32, more than 128 latents): the dQ accumulators of all latents would take more than 64 registers, so two
    // waves share a token tile, each with half of the latent tiles.  At the end of the tile the first hands its part of dK
    // to the second and takes that one's part of dV (16 values a lane, through the dS tiles, which are free by then); the
    // two wait for each other by counters in LDS (lds_post, lds_wait), not at a barrier of the workgroup, which would bring
    // all eight waves into step.  Every wait ends: both waves are in the workgroup, and they take the same token tiles, since
    // `tile` and `stride` depend on wave >> 1 only.  (262144 tokens, 8 heads, 256 latents: a dQ kernel of its own 283 us and dK/dV 235, this one 320; 32 x 8
    // heads, 4096 tokens, 128 latents without PAIR: training 316 -> 248 us.)
    constexpr bool PAIR = DQ && dkdv_pair(D, MT);
    static_assert(!PAIR || MT % 2 == 0, "the latent tiles are halved");
    constexpr int HT = PAIR ? MT / 2 : MT;      // latent tiles of a wave
    constexpr int TW = PAIR ? WV / 2 : WV;      // token tiles a workgroup works on at a time
    constexpr int DB = D / 16;                  // 16-row blocks of the dQ product
    constexpr int kKtStride = kt_stride(D);
    // ZL (DQ at d = 16, shapes with fewer tokens than latents): the c chain carries the lo term of Z as one more image
    // and product (at d <= 8 it rides in the free upper half of the Z image, ZPACK below).  dQ sums dS over the tokens
    // of one latent, so the rounding of Z_m adds up coherently there, and on rows whose halves cancel it shows:
    // mesh-like inputs, 692 latents over 242 tokens, dq_lat 2.4e-2 without it, 1.1e-2 with it (1539 over 427: 2.5e-2
    // and 7e-3).  It costs 5 % of the kernel's time; of the random shapes with at least as many tokens as latents one
    // in 30 000 left the bar, and that one for another reason (delta from the saved bf16 y), the lo term or not.
    constexpr bool ZLO = DQ && !pack_dim(DR) && ZL;
    static_assert(!ZL || (DQ && !pack_dim(DR)), "the extra image is for the fused dQ product at d = 16");
    constexpr int NA = dkdv_a_images(DR, DQ, ZL), PER_TILE = dkdv_images(DR, DQ, ZL);
    constexpr int NR = 4 * HV;                  // row images per latent tile (RW1, RW2) x 2 k-steps
    static_assert(PER_TILE == NA + NR && ZLO == (NA == 5 * KS + 1), "as counted");
    constexpr bool PIPE = (D == 16);            // look one latent tile ahead where registers allow
    // d <= 8: the upper half of the padded contraction carries what otherwise needs products of its own.
    // Images: q' hi | lo in one (keys repeated in both lane halves), slots 8,9 of the dZ image = -eps
    // (against ones in the V operand), slots 8,9 of the Z image = 1, 1 (against -delta in
    // the dY operand).  The q' lo image and the a / c parts of the correction image are then unused.
    constexpr bool PACK = pack_dim(DR);
    // PACK with DQ: the upper half of the Z image carries the lo term of Z instead (dY rows repeated in both
    // lane halves), as the separate dQ kernel has it at d <= 8, and -delta comes in through the correction
    // image as at d = 16: dQ sums dS over the tokens of one latent, and with so few terms per dot product
    // the rounding of Z_m showed (9.7e-3 against 2.6e-3 on a 1500-token case).  The delta it subtracts
    // comes from rows of Y formed with the same hi + lo pair (the token-statistics kernel at d <= 8), so
    // c - delta cancels where one latent dominates a token, down to a single latent.
    constexpr bool ZPACK = PACK && DQ;
    // ... and with one exponential, where dS = P (a + w c) and a takes both corrections, -w delta comes in through slots 10, 11 of
    // the dZ image (ones, against the hi + lo pair in the V operand) beside -eps: no correction product at all.
    constexpr bool APACK = ZPACK && ONE;
    extern __shared__ __attribute__((aligned(16))) u32x4 img[];   // [MT][PER_TILE][64 lanes]
    __shared__ int posted[PAIR ? WV : 1], taken[PAIR ? WV : 1];   // PAIR: parts handed over / picked up so far

    const int tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // known to be wave-uniform: scalar unit
    const GridPos gp = grid_pos_latents(ts, H, DR * 2);
    const int bh = gp.y, h = bh % H;
    const bool lower = hh == 0;
    constexpr float kap = 0.f;                  // w[n] = 2^(kap - lse_dec2[n])

    if constexpr (PAIR) {
        if (tid < WV) { posted[tid] = 0; taken[tid] = 0; }
    }
    const bf16_t *kb = k + tok_base(ts, bh, H);
    const bf16_t *vb = v + tok_base(ts, bh, H);
    const bf16_t *gb = dy + tok_base(ts, bh, H);
    const float *lb = lse_dec2 + (size_t)bh * N;
    const float *db = delta + (size_t)bh * N;
    const int tiles = (N + 31) / 32;
    const int stride = gridDim.x * TW;
    const int half = PAIR ? wave & 1 : 0;
    // B operand: column = token.  rep (PACK only): both lane halves get elements 0-7 of the row.
    auto load_cols = [&](const bf16_t *base, int tile, bf16x8 (&t)[KS], bool rep) {
        const int n = min(tile * 32 + l32, N - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s)
            t[s] = as_bf16x8(row8_bf16<DR>(base + tok_off(ts, n), (PACK && rep) ? 0 : (D / 2) * hh + 8 * s));
    };
    // The first token tile's rows and statistics are requested before the operand images are built.
    int tile = gp.x * TW + (PAIR ? wave >> 1 : wave);
    bf16x8 kt[KS], vt[KS], gt[KS], ktn[KS], vtn[KS], gtn[KS];
    float lse_next = 0.f, delta_next = 0.f;
    if (tile < tiles) {
        load_cols(kb, tile, kt, true);
        load_cols(vb, tile, vt, false);
        load_cols(gb, tile, gt, ZPACK);
        const size_t row0 = (size_t)min(tile * 32 + l32, N - 1);
        lse_next = lb[row0];
        delta_next = db[row0];
    }
    // ---- build the operand images ----
    {
        // DQ: the latents' rows of q and z and their lse_enc were staged in the waves' part of the LDS (LatentPieces), from where
        // every image takes its own elements; dz, eps: the rows of this (b,h), in global memory or merged into LDS.
        const LatentStage<DR> st(img + MT * PER_TILE * 64, mend - m0);
        const bf16_t *qh_ = DQ ? st.q : q + (size_t)h * ts.sq + (size_t)m0 * DR;
        const float *zb = DQ ? st.z : z + ((size_t)bh * Mtot + m0) * DR;
        const float *leb = DQ ? st.lse : lse_enc + (size_t)bh * Mtot + m0;
        const float *dzb = dz + (size_t)m0 * DR;
        const float *eb = eps + m0;
        // Padding latents (at or beyond mend; mleft = real ones from m0 on): reads are clamped to the last
        // real latent and every value that could reach dK or dV is zero -- q, Z, dZ, eps, u and the ones
        // that pick -delta -- so that a = c = 0 and dS = 0 whatever P and R come out as.
        const int mleft = mend - m0;
        // all ones where a < b (as a value: the results of many compares side by side take the scalar registers that the token loop
        // needs, and every one spilled there costs it vector registers)
        auto below = [](int a, int b) { return (uint32_t)((a - b) >> 31); };
        // A wave makes the images of one kind for GT latent tiles at a time: which kind it is, is the same for all its lanes, and the
        // tiles' reads wait together.  (All tiles together: kinds do not divide evenly over the waves, and at eight tiles 200 scalar
        // registers spilled.  An image at a time, 2 x 8 heads, 7225 tokens, 100 latents, d = 16: 19.9 us the kernel, 18.2 so.)
        constexpr int GT = MT < 2 ? 1 : 2, GROUPS = (MT + GT - 1) / GT;
#pragma unroll 1
        for (int u = wave; u < PER_TILE * GROUPS; u += WV) {
            const int sid = u / GROUPS, t0 = u % GROUPS * GT;
            u32x4 im[GT];
            if (sid == NA - 1) {
                // correction operand: slots 0,1 = -lse_enc2 (hi + lo pair), slots 2,3 = 1, else zero
                // Slots 4,5 and 8-11 belong to the a and c products, whose operands are bf16
                // whatever the storage type; the score products meet them with zeros in the token operand
                // (and the a and c products meet slots 0-3 with zeros).  Finite 16-bit patterns of either type read as
                // finite values of the other, so the foreign slots contribute exact zeros.
#pragma unroll
                for (int t = 0; t < GT; ++t) {
                    const int m = 32 * (t0 + t) + l32, mc = min(m, mleft - 1);
                    const uint32_t real = below(m, mleft);
                    u32x4 &w = im[t];
                    w[0] = lower ? split_pair<F>(-(leb[mc] * kLog2e)) & real
                                 : split_bf16_pair(-eb[mc]) & real;             // slots 8,9 := -eps (bf16: the a chain)
                    w[1] = lower ? kOnePair<F> : ONE ? 0u : 0x3f803f80u & real;   // slots 10,11 := 1 (picks -delta, two exponentials)
                    // one exponential: slots 4,5 := 1 (they pick -w delta hi, lo; the latent's factor of the c chain is 1)
                    w[2] = ONE && lower ? 0x3f803f80u & real : 0u;
                    w[3] = 0u;
                }
            } else if (sid < NA) {
                const int kind = sid / KS, ks = sid % KS;          // 0 q' hi, 1 q' lo, 2 dZ, 3 Z hi, 4 Z lo (DQ only)
                const int d0 = (D / 2) * hh + 8 * ks;
                const bool want_lo = kind == 1 || kind >= 4 || (!lower && ((PACK && kind == 0) || (ZPACK && kind == 3)));
                const uint32_t take_lo = want_lo ? 0xffffffffu : 0u;
                if (kind <= 1) {
#pragma unroll
                    for (int t = 0; t < GT; ++t) {
                        const int m = 32 * (t0 + t) + l32;
                        const uint32_t real = below(m, mleft);
                        const u32x4 raw = row8_bf16<DR>(qh_ + (size_t)min(m, mleft - 1) * DR, PACK ? 0 : d0);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {              // q' feeds the score products: storage type
                            const HiLo p = split_scaled<F>(raw[i], c2);
                            im[t][i] = ((p.lo & take_lo) | (p.hi & ~take_lo)) & real;
                        }
                    }
                } else {
                    const float *src = kind == 2 ? dzb : zb;
                    const int e0 = ZPACK && kind >= 3 ? 0 : d0;
#pragma unroll
                    for (int t = 0; t < GT; ++t) {
                        const int m = 32 * (t0 + t) + l32, mc = min(m, mleft - 1);
                        const uint32_t real = below(m, mleft);
                        float x[8];
                        row8_f32<DR>(src + (size_t)mc * DR, e0, x);
                        u32x4 &w = im[t];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const HiLo p = split_elems<false>(x[2 * i], x[2 * i + 1]);
                            w[i] = ((p.lo & take_lo) | (p.hi & ~take_lo)) & real;
                            if constexpr (DR == 4 && !ZPACK) {   // slots 4-7 of the Z image := its lo part (dY repeated there)
                                if (kind == 3 && i >= 2) w[i] = lower ? split_elems<false>(x[2 * i - 4], x[2 * i - 3]).lo & real : 0u;
                            }
                        }
                        if (PACK && !lower && kind == 2) {
                            w[0] = split_bf16_pair(-eb[mc]) & real;                    // slots 8,9 := -eps
                            if constexpr (APACK) w[1] = 0x3f803f80u & real;            // slots 10,11 := 1 (pick -w delta)
                        }
                        if (PACK && !ZPACK && !lower && kind == 3) w[0] = 0x3f803f80u & real;   // slots 8,9 := 1 (pick -delta)
                    }
                }
            } else {
                const int rsid = sid - NA;                          // (which, hv, s2)
                const int which = rsid / (2 * HV), hv = (rsid / 2) % HV, s2 = rsid % 2;
                const int dd = WIDE ? l32 : 16 * hv + (l32 & 15);
                // beyond the real head dimension every row image is zero
                const uint32_t keep = (WIDE || l32 < 16) && dd < DR ? 0xffffffffu : 0u;
                const int dc = dd & (DR - 1);
#pragma unroll
                for (int t = 0; t < GT; ++t) {
#pragma unroll
                    for (int i = 0; i < 8; i += 2) {
                        const int ma = 32 * (t0 + t) + perm_index(s2, hh, i), mb = ma + 1;
                        const int ca = min(ma, mleft - 1) * DR + dc, cb = min(mb, mleft - 1) * DR + dc;
                        uint32_t x;
                        if (which == 0) x = cvt_pk_bf16(dzb[ca], dzb[cb]);
                        else if constexpr (F) x = cvt_pk_bf16(elem_value<F>(qh_[ca]), elem_value<F>(qh_[cb]));
                        else x = (uint32_t)qh_[ca] | ((uint32_t)qh_[cb] << 16);
                        im[t][i / 2] = x & keep & ((below(ma, mleft) & 0xffffu) | (below(mb, mleft) << 16));
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < GT; ++t)
                if (t0 + t < MT) img[((t0 + t) * PER_TILE + sid) * 64 + lane] = im[t];
        }
    }
    __syncthreads();

    u32x4 w11;
    w11[1] = 0u; w11[2] = 0u; w11[3] = 0u;
    w11[0] = lower ? kOnePair<F> : 0u;
    const bf16x8 ones_s = as_bf16x8(w11);        // the same in the type of the score products
    w11[0] = lower ? 0u : 0x3f803f80u;
    const bf16x8 ones_eps = as_bf16x8(w11);      // slots 8,9 = 1 (bf16): picks -eps out of the correction image
    auto to_bf16 = [](bf16x8 x) { return as_bf16x8(to_bf16_row<F>(__builtin_bit_cast(u32x4, x))); };

    // V rows as the operand of the a product; PACK: slots 8,9 := 1 (the upper lane half loaded zeros)
    auto v_operand = [&](bf16x8 x) {
        u32x4 w = to_bf16_row<F>(__builtin_bit_cast(u32x4, x));
        if (PACK && !lower) w[0] = 0x3f803f80u;
        return as_bf16x8(w);
    };
    // t: of this wave's latent tiles.  (As an index: a pointer to the wave's first image took two registers more also where
    // half is the constant 0, and the d = 16 kernel of six tiles spilled: two exponentials, 131072 tokens, 8 heads, 336
    // latents 230 us, 213 like this.)
    auto image = [&](int t, int sid) { return as_bf16x8(img[((half * HT + t) * PER_TILE + sid) * 64 + lane]); };

    // fused dQ: wave-private LDS tiles and the accumulators dQ^T[dd = 16 db + 4 (lane / 16) + r][m = 32 t + 16 jb + lane % 16]
    uint16_t *ds_t = reinterpret_cast<uint16_t *>(img + MT * PER_TILE * 64) + (DQ ? wave * fused_wave_lds(D, MT) : 0);
    uint16_t *k_t = ds_t + ds_tile_lds(D, MT);
    if constexpr (DQ && PACK) {   // columns 8-15 of the key tile are never written at d <= 8: zero (the output rows 8-15 are dropped)
        if (lane < 32) *reinterpret_cast<u32x4 *>(k_t + lane * kKtStride + 8) = u32x4{0u, 0u, 0u, 0u};
    }
    f32x4 dqa[DQ ? HT : 1][2][DB];
#pragma unroll
    for (int t = 0; t < (DQ ? HT : 1); ++t)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int db = 0; db < DB; ++db) dqa[t][jb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int c16 = lane & 15, g16 = lane >> 4;

    int round = 0;   // PAIR: token tiles so far
    if (tile < tiles) {
#pragma unroll
        for (int s = 0; s < KS; ++s) { vt[s] = v_operand(vt[s]); gt[s] = to_bf16(gt[s]); }
    }
    // The token statistics (lse_dec2, delta) are requested one tile ahead like the rows: a request made where its
    // value is needed would also wait for the rows requested just before it (loads complete in order), and every
    // token tile would begin with a full memory latency.
    // (the first tile's rows and statistics have arrived before the loop starts: inside it, nothing waits for
    // anything but what the loop itself requested a tile earlier)
    float nld_cur = pinned(-lse_next * ld_mul), dl_cur = pinned(delta_next);
#pragma unroll
    for (int s = 0; s < KS; ++s) { kt[s] = pinned(kt[s]); vt[s] = pinned(vt[s]); gt[s] = pinned(gt[s]); }
    for (; tile < tiles; tile += stride) {
        const int n = tile * 32 + l32;
        const int tn = (tile + stride < tiles) ? tile + stride : tile;
        load_cols(kb, tn, ktn, true);
        load_cols(vb, tn, vtn, false);
        load_cols(gb, tn, gtn, ZPACK);
        const float nld = nld_cur, dl = dl_cur;
        {
            const size_t rown = (size_t)min(tn * 32 + l32, N - 1);
            lse_next = lb[rown];
            delta_next = db[rown];
        }
        const float wn = ONE ? fast_exp2(kap + nld) : 0.f;

        u32x4 wb;
        wb[0] = 0u; wb[2] = 0u; wb[3] = 0u;
        wb[1] = lower ? split_pair<F>(nld) : 0u;             // slots 2,3 := -lse_dec2[n]
        const bf16x8 kt_a = ones_s, kt_b = as_bf16x8(wb);    // slots 0,1 := 1 picks -lse_enc2
        // Token side of the correction k-step(s).  Two exponentials: g_aug picks -delta for the c chain
        // (slots 10,11 against the image's ones) and ones_eps picks -eps for the a chain.  One exponential:
        // dS = P (a + w c), and w[n] is this lane's scalar, so one product carries both corrections: slots 8,9 = 1
        // pick -eps and slots 4,5 = -w delta (hi, lo) meet ones; the a chain starts from it and the c chain from
        // zero.  (d <= 8: the operands' free slots carry them, see PACK, ZPACK and APACK.)
        u32x4 wg;
        const uint32_t ds_ = split_bf16_pair(ONE ? -dl * wn : -dl);
        wg[0] = (ONE && !lower && !PACK) ? 0x3f803f80u : 0u;
        wg[1] = (!ONE && !lower) ? ds_ : 0u;                 // two exponentials: slots 10,11 := -delta (hi, lo)
        wg[2] = (ONE && lower) ? ds_ : 0u;                   // one: slots 4,5 := -w delta (hi, lo)
        wg[3] = 0u;
        const bf16x8 g_aug = as_bf16x8(wg);
        if constexpr (APACK) {   // slots 10,11 of the V operand := -w delta hi, lo
            u32x4 w = __builtin_bit_cast(u32x4, vt[0]);
            w[1] = lower ? w[1] : ds_;
            vt[0] = as_bf16x8(w);
        }
        bf16x8 gc[KS];   // dY operand of the c product; PACK without dQ: slots 8,9 := -delta (hi, lo)
#pragma unroll
        for (int s = 0; s < KS; ++s) gc[s] = gt[s];
        if constexpr (PACK && !ZPACK) {
            u32x4 w = __builtin_bit_cast(u32x4, gt[0]);
            const uint32_t dp_ = split_bf16_pair(-dl);   // here c keeps its own correction: -delta unscaled
            if (!lower) { w[0] = dp_; w[1] = 0u; }
            if (DR == 4 && lower) { w[2] = w[0]; w[3] = w[1]; }   // against the lo part of Z in slots 4-7
            gc[0] = as_bf16x8(w);
        }

        f32x16 acc1[HV], acc2[HV];
#pragma unroll
        for (int hv = 0; hv < HV; ++hv) { acc1[hv] = splat16(0.f); acc2[hv] = splat16(0.f); }

        // fused dQ: K^T of this token tile as the A operand of the 16x16x32 product (row = dd = lane % 16,
        // tokens 8 (lane / 16) .. + 7), through the wave's LDS tile; rows of tokens past N are zero
        bf16x8 k_op[DB];
        if constexpr (DQ) {
            // the tile as loaded, row = token (one 16-byte store per lane and k-step); the transposing read hands lane c16 of
            // block g16 column c16 of the rows 8 g16 .. + 3 (second read: + 4 .. + 7), as for the dS tile below
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const u32x4 w = (n < N) ? to_bf16_row<F>(__builtin_bit_cast(u32x4, kt[s])) : __builtin_bit_cast(u32x4, zero_operand());
                if (!(PACK && hh))     // d <= 8: the upper lane half holds a copy of the same elements
                    *reinterpret_cast<u32x4 *>(k_t + l32 * kKtStride + (D / 2) * hh + 8 * s) = w;
            }
            compiler_fence();
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint16_t *src = k_t + (8 * g16 + c16 / 4) * kKtStride + 16 * db + 4 * (c16 % 4);
                const u32x2 lo2 = lds_read_tr16(src), hi2 = lds_read_tr16(src + 4 * kKtStride);
                k_op[db] = as_bf16x8(u32x4{lo2[0], lo2[1], hi2[0], hi2[1]});
            }
        }

        // Score products of latent tile t (minus lse_enc2 / minus lse_dec2): 2*KS + 2 MFMAs.
        auto scores = [&](int t, f32x16 &s1, f32x16 &s2) {
            f32x16 x = splat16(0.f);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) x = mfma_s<F>(image(t, 0 * KS + ks), kt[ks], x);
            if constexpr (!PACK) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) x = mfma_s<F>(image(t, 1 * KS + ks), kt[ks], x);
            }
            if constexpr (ONE) {
                s1 = x;                         // one exponential: the scores as they are
            } else {
                const bf16x8 qa = image(t, NA - 1);
                s1 = mfma_s<F>(qa, kt_a, x);
                s2 = mfma_s<F>(qa, kt_b, x);
            }
        };
        // One latent tile, software-pipelined: the a and c products of tile t and the score products
        // of tile t+1 are issued first and run on the matrix cores while the vector ALUs
        // exponentiate the scores of tile t (s1, s2, computed one step earlier).
        auto tile_step = [&](int t, f32x16 &s1, f32x16 &s2, f32x16 &s1n, f32x16 &s2n) {
            // The wave takes issue priority over its SIMD's other wave while it feeds the matrix cores (the a and
            // c products, the next tile's scores) and drops it for the vector block: the matrix pipe starts
            // at once and the other wave's vector instructions fill the gaps (measured -4.5 % at d = 16, -2 to
            // -6 % at the other shapes; holding the priority over the accumulation products as well was
            // slower, and the same switch in the encode kernel changed nothing, in the dQ kernel it cost 5 %).
            __builtin_amdgcn_s_setprio(1);
            if constexpr (!PIPE) scores(t, s1, s2);   // not enough registers at d = 32: no look-ahead
            f32x16 av = splat16(0.f), cv = splat16(0.f);
            if constexpr (ONE) {
                if constexpr (!PACK) av = mfma(image(t, NA - 1), g_aug, av);
            } else {
                if constexpr (!PACK) av = mfma(image(t, NA - 1), ones_eps, av);
                if constexpr (!PACK || ZPACK) cv = mfma(image(t, NA - 1), g_aug, cv);
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                av = mfma(image(t, 2 * KS + ks), vt[ks], av);
                cv = mfma(image(t, 3 * KS + ks), gc[ks], cv);
                if constexpr (ZLO) cv = mfma(image(t, 4 * KS + ks), gc[ks], cv);
            }
            if constexpr (PIPE) {
                if (t + 1 < HT) scores(t + 1, s1n, s2n);
            }
            // Two exponentials at d = 32: both scores, a and c are 64 registers, and with the row images beside them 26 to 39
            // others were spilled and read again in every latent tile.  So these come behind the vector block there (0 to 4
            // spilled): 131072 tokens, 8 heads, 128 latents 167 -> 109 us, 256 latents 280 -> 194 (with a dQ kernel of its
            // own 174 and 293).
            constexpr bool LATE_ROWS = WIDE && !ONE;
            bf16x8 rw[NR];
            if constexpr (!LATE_ROWS) {
#pragma unroll
                for (int r = 0; r < NR; ++r) rw[r] = image(t, NA + r);
            }
            sched_fence();
            __builtin_amdgcn_s_setprio(0);
            f32x16 pv, rv;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                pv[i] = fast_exp2(s1[i]);
                if constexpr (ONE) rv[i] = pv[i] * fmaf(cv[i], wn, av[i]);     // dS' = P (a + w[n] u[m] c)
                else rv[i] = fmaf(fast_exp2(s2[i]), cv[i], pv[i] * av[i]);     // dS' = P a + R c
            }
            u32x4 p0, p1, d0, d1;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                p0[i] = cvt_pk_bf16(pv[2 * i], pv[2 * i + 1]);
                p1[i] = cvt_pk_bf16(pv[8 + 2 * i], pv[8 + 2 * i + 1]);
                d0[i] = cvt_pk_bf16(rv[2 * i], rv[2 * i + 1]);
                d1[i] = cvt_pk_bf16(rv[8 + 2 * i], rv[8 + 2 * i + 1]);
            }
            if constexpr (LATE_ROWS) {
                sched_fence();
#pragma unroll
                for (int r = 0; r < NR; ++r) rw[r] = image(t, NA + r);
            }
#pragma unroll
            for (int hv = 0; hv < HV; ++hv) {
                acc1[hv] = mfma(rw[(0 * HV + hv) * 2 + 0], as_bf16x8(p0), acc1[hv]);
                acc1[hv] = mfma(rw[(0 * HV + hv) * 2 + 1], as_bf16x8(p1), acc1[hv]);
                acc2[hv] = mfma(rw[(1 * HV + hv) * 2 + 0], as_bf16x8(d0), acc2[hv]);
                acc2[hv] = mfma(rw[(1 * HV + hv) * 2 + 1], as_bf16x8(d1), acc2[hv]);
            }
            if constexpr (DQ) {
                // dS (this lane: token l32, latents 8 (r/4) + 4 hh + r%4 for r = 0..15) -> LDS as it is, row = token:
                // four 8-byte stores of four latents each.  The product wants it the other way round (column =
                // latent, 8 consecutive tokens per lane): four transposing reads, each four tokens of one latent.
                if constexpr (PAIR) {   // the other wave has what was left here at the end of the tile before
                    if (t == 0) lds_wait(taken + (wave ^ 1), round);
                }
                uint16_t *drow = ds_t + l32 * kDsStride + 4 * hh;
                *reinterpret_cast<u32x2 *>(drow) = u32x2{d0[0], d0[1]};
                *reinterpret_cast<u32x2 *>(drow + 8) = u32x2{d0[2], d0[3]};
                *reinterpret_cast<u32x2 *>(drow + 16) = u32x2{d1[0], d1[1]};
                *reinterpret_cast<u32x2 *>(drow + 24) = u32x2{d1[2], d1[3]};
                compiler_fence();
#pragma unroll
                for (int jb = 0; jb < 2; ++jb) {
                    // lane c16 of block g16: chunk row = token 8 g16 (+ 4) + c16 / 4, piece = latents 16 jb + 4 (c16 % 4)
                    const uint16_t *src = ds_t + (8 * g16 + c16 / 4) * kDsStride + 16 * jb + 4 * (c16 % 4);
                    const u32x2 b_lo = lds_read_tr16(src), b_hi = lds_read_tr16(src + 4 * kDsStride);
                    const u32x4 bop = u32x4{b_lo[0], b_lo[1], b_hi[0], b_hi[1]};
#pragma unroll
                    for (int db = 0; db < DB; ++db)
                        dqa[t][jb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_op[db], as_bf16x8(bop), dqa[t][jb][db], 0, 0, 0);
                }
                compiler_fence();
            }
            // (the fused one-exponential kernel of d = 16 is 0.6 % faster without this fence between its latent tiles)
            if constexpr (!(DQ && ONE && D == 16)) sched_fence();
        };
        {
            f32x16 sa1 = splat16(0.f), sa2 = splat16(0.f), sb1 = splat16(0.f), sb2 = splat16(0.f);
            if constexpr (PIPE) scores(0, sa1, sa2);
            if constexpr (HT == 1) {
                tile_step(0, sa1, sa2, sb1, sb2);
            } else if constexpr (DQ) {   // unrolled: the dQ accumulators are indexed by the latent tile
#pragma unroll
                for (int t = 0; t + 1 < HT; t += 2) {
                    tile_step(t, sa1, sa2, sb1, sb2);
                    tile_step(t + 1, sb1, sb2, sa1, sa2);
                }
                if constexpr (HT % 2 != 0) tile_step(HT - 1, sa1, sa2, sb1, sb2);
            } else {
#pragma unroll 1
                for (int t = 0; t + 1 < MT; t += 2) {
                    tile_step(t, sa1, sa2, sb1, sb2);
                    tile_step(t + 1, sb1, sb2, sa1, sa2);
                }
                if constexpr (MT % 2 != 0) tile_step(MT - 1, sa1, sa2, sb1, sb2);
            }
        }
        if constexpr (PAIR) {
            // [4][64 lanes] float4: the part that the other wave finishes
            float4 *give = reinterpret_cast<float4 *>(ds_t) + lane;
            const f32x16 &part = half ? acc1[0] : acc2[0];
            compiler_fence();
#pragma unroll
            for (int i = 0; i < 4; ++i)
                give[64 * i] = make_float4(part[4 * i], part[4 * i + 1], part[4 * i + 2], part[4 * i + 3]);
            lds_post(posted + wave, ++round, lane);
        }
        // What was requested at the top of this tile is taken over here, ahead of the tile's stores: memory
        // operations complete in order, so taking it over after them (at the top of the next tile) would make the
        // wave wait for its own stores once per tile.
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kt[s] = pinned(ktn[s]);
            vt[s] = pinned(v_operand(vtn[s]));
            gt[s] = pinned(to_bf16(gtn[s]));
        }
        nld_cur = pinned(-lse_next * ld_mul);
        dl_cur = pinned(delta_next);
        compiler_fence();
        if constexpr (PAIR) {
            lds_wait(posted + (wave ^ 1), round);
            const float4 *get = reinterpret_cast<const float4 *>(ds_t + (1 - 2 * half) * fused_wave_lds(D, MT)) + lane;
            f32x16 &mine = half ? acc2[0] : acc1[0];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 o = get[64 * i];
                mine[4 * i] += o.x; mine[4 * i + 1] += o.y; mine[4 * i + 2] += o.z; mine[4 * i + 3] += o.w;
            }
            lds_post(taken + wave, round, lane);
        }
        const bool has_dv = !PAIR || half == 0, has_dk = !PAIR || half != 0;
        // registers 4 q .. 4 q + 3 of an accumulator: columns (16 hv +) 8 q + 4 hh .. + 3 of this lane's token
        // More than one latent chunk: all but the first add what the chunks before them left in acc32, and all but
        // the head's last one leave their sums there; the last one rounds and stores them like a single chunk.
        const bool from_acc = acc32 != nullptr && m0 != 0;
        const bool to_acc = acc32 != nullptr && mend < Mtot;
        if (n < N) {
#pragma unroll
            for (int hv = 0; hv < HV; ++hv)
#pragma unroll
                for (int qd = 0; qd < QUARTS; ++qd) {
                    const int o = 16 * hv + 8 * qd + 4 * hh;
                    if (o >= DR) continue;
                    float4 a = make_float4(acc1[hv][4 * qd], acc1[hv][4 * qd + 1], acc1[hv][4 * qd + 2],
                                           acc1[hv][4 * qd + 3]);
                    float4 b = make_float4(scale * acc2[hv][4 * qd], scale * acc2[hv][4 * qd + 1],
                                           scale * acc2[hv][4 * qd + 2], scale * acc2[hv][4 * qd + 3]);
                    if (from_acc || to_acc) {
                        float *dvr = acc32 + ((size_t)bh * N + n) * DR + o;
                        float *dkr = dvr + (size_t)gridDim.y * N * DR;
                        if (from_acc) {
                            if (has_dv) add4(a, *reinterpret_cast<const float4 *>(dvr));
                            if (has_dk) add4(b, *reinterpret_cast<const float4 *>(dkr));
                        }
                        if (to_acc) {
                            if (has_dv) *reinterpret_cast<float4 *>(dvr) = a;
                            if (has_dk) *reinterpret_cast<float4 *>(dkr) = b;
                        }
                    }
                    if (!to_acc) {
                        const size_t at = tok_base(ts, bh, H) + tok_off(ts, n) + o;
                        u32x2 w;
                        if (has_dv) {
                            w[0] = pack_elems<F>(a.x, a.y);
                            w[1] = pack_elems<F>(a.z, a.w);
                            *reinterpret_cast<u32x2 *>(dv + at) = w;
                        }
                        if (has_dk) {
                            w[0] = pack_elems<F>(b.x, b.y);
                            w[1] = pack_elems<F>(b.z, b.w);
                            *reinterpret_cast<u32x2 *>(dk + at) = w;
                        }
                    }
                }
        }
    }

    if constexpr (DQ) {
        // The waves' dQ partials are added in wave order (fixed, so the bits are reproducible) and the workgroup stores its slot:
        // as many latent tiles at a time as fit the LDS of images and waves once for every wave (one to three rounds; one wave
        // after the other adding to a single sum took 4 us at 128 latents and d = 32).
        // (the lane counted anew: what is kept from before the token loop costs that a register)
        const int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        float *red = reinterpret_cast<float *>(img);
        constexpr int kTileFloats = 32 * D;                      // of one wave
        constexpr int kFit = (MT * PER_TILE * 1024 + WV * fused_wave_lds(D, MT) * 2) / (WV * kTileFloats * 4);
        static_assert(kFit >= 1, "the images and the waves' tiles leave room for one latent tile of every wave");
        constexpr int kRounds = (HT + kFit - 1) / kFit, TB = (HT + kRounds - 1) / kRounds;   // latent tiles (of a wave) a round
        constexpr int STEP = PAIR ? 2 : 1;                       // (the two halves of the latents side by side)
        const int mleft = mend - m0;
        float *out = dq_part + (((size_t)bh * gridDim.x + gp.x) * Mtot + m0) * DR;
        constexpr int PCS = DR / 4;                              // float4 pieces of a DR-element row
#pragma unroll
        for (int t0 = 0; t0 < HT; t0 += TB) {
            __syncthreads();   // every wave is done with the images, or with the round before
#pragma unroll
            for (int t = t0; t < t0 + TB && t < HT; ++t)
#pragma unroll
                for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        const f32x4 &q4 = dqa[t][jb][db];
                        *reinterpret_cast<float4 *>(red + (wave * TB + t - t0) * kTileFloats + (16 * jb + (ln & 15)) * D + 16 * db + 4 * (ln >> 4)) =
                            make_float4(q4[0], q4[1], q4[2], q4[3]);
                    }
            __syncthreads();
            for (int i = 64 * wave + ln; i < STEP * TB * 32 * PCS; i += 64 * WV) {
                const int pc = i % PCS, r = i / PCS, hf = STEP == 1 ? 0 : r / (32 * TB), row = r - hf * 32 * TB;
                const int lat = 32 * (hf * HT + t0) + row;
                const float *src = red + (hf * TB * 32 + row) * D + 4 * pc;
                float4 x = *reinterpret_cast<const float4 *>(src);
#pragma unroll
                for (int w = 1; w < WV / STEP; ++w) add4(x, *reinterpret_cast<const float4 *>(src + w * STEP * TB * kTileFloats));
                if (t0 + row / 32 < HT && lat < mleft) *reinterpret_cast<float4 *>(out + (size_t)lat * DR + 4 * pc) = x;
            }
        }
    }
}

#define FLARE_DKDV_PARAMS                                                                                        \
    const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,                    \
        const bf16_t *__restrict__ dy, const float *__restrict__ z, const float *__restrict__ lse_enc,           \
        const float *__restrict__ lse_dec2, const float *__restrict__ delta, float ld_mul, bf16_t *__restrict__ dk, \
        bf16_t *__restrict__ dv, float *__restrict__ acc32, float *__restrict__ dq_part, TokStride ts, int H,    \
        int N, int Mtot, int m0, int mend, float c2, float scale, MergeDz merge
#define FLARE_DKDV_PASS \
    q, k, v, dy, z, lse_enc, dz_bh, eps_bh, lse_dec2, delta, ld_mul, dk, dv, acc32, dq_part, ts, H, N, Mtot, m0, mend, c2, scale

// Both variants in one launch, each workgroup taking the one that the plan names for its (b,h): one launch less per step
// (a launch whose workgroups all leave at once still costs 4-6 us).  Both bodies share the kernel's registers,
// which at one workgroup per CU costs nothing.
template <int DR, int MT, bool DQ, bool F, bool ZL = false>
__global__ __launch_bounds__(64 * WV, 1) void bwd_dkdv_planned_kernel(FLARE_DKDV_PARAMS)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 img[];
    __shared__ float red[64];
    const GridPos gp = grid_pos_latents(ts, H, DR * 2);
    float *rows = reinterpret_cast<float *>(reinterpret_cast<char *>(img) + merge.lds);
    const float *dz_bh, *eps_bh;
    LatentPieces<DR, DQ ? MT : 0> pieces;
    if constexpr (DQ) {
        const size_t row = (size_t)gp.y * Mtot + m0;
        pieces.request(q + (size_t)(gp.y % H) * ts.sq + (size_t)m0 * DR, z + row * DR, lse_enc + row, mend - m0);
    }
    auto put = [&]() {
        if constexpr (DQ) pieces.put(img + MT * dkdv_images(DR, DQ, ZL) * 64, mend - m0);
    };
    // (a dQ kernel of its own runs behind this one and reads what workgroup 0 writes)
    const bool one = merged_dz<DR>(merge, z, lse_enc, gp.y, Mtot, true, !DQ && gp.x == 0, rows, red, dz_bh, eps_bh, put);
    if (DQ && merge.parts == 0) __syncthreads();     // (merging has barriers of its own)
    if (one)
        dkdv_body<DR, MT, DQ, true, F, ZL>(FLARE_DKDV_PASS);
    else
        dkdv_body<DR, MT, DQ, false, F, ZL>(FLARE_DKDV_PASS);
}
#undef FLARE_DKDV_PASS
#undef FLARE_DKDV_PARAMS

}  // namespace

// dQ partials of the backward; slot layout as the encode partials: [(b*h) * parts + part][M][d]
int mfma_dq_partial(const flare_shape &s, const void *q, const void *k, const void *v, const void *dy,
                    const float *z, const float *lse_enc, const float *dz, const float *eps,
                    const float *lse_dec2, const float *delta, float ld_mul, const int *plan, float *dq_part,
                    float scale, hipStream_t stream)
{
    const MfmaPlan p = mfma_plan(s);
    const EncGeom e = dq_geom(s);
    const int BH = s.B * s.H;
    const float c2 = scale * kLog2e;
    const int parts = p.enc.chunks * e.TG;
    const dim3 grid(p.enc.chunks, BH, e.Z);
    const bf16_t *qq = (const bf16_t *)q, *kk = (const bf16_t *)k, *vv = (const bf16_t *)v, *gg = (const bf16_t *)dy;
    LaunchTimer t(KID_BWD_DQ_PARTIAL, stream);
    const bool f16 = s.dtype == FLARE_F16;
#define FLARE_DQ_ARGS                                                                                            \
    qq, kk, vv, gg, z, lse_enc, dz, eps, lse_dec2, delta, ld_mul, plan, dq_part, tok_stride(s), s.H, s.N, s.M,   \
        p.enc.chunk_len, parts, e.G, e.TG, c2
#define FLARE_DQ(DD, NBB, MINB)                                                                                  \
    do {                                                                                                         \
        if (f16) bwd_dq_mfma_kernel<DD, NBB, MINB, true><<<grid, e.threads, 0, stream>>>(FLARE_DQ_ARGS);         \
        else bwd_dq_mfma_kernel<DD, NBB, MINB, false><<<grid, e.threads, 0, stream>>>(FLARE_DQ_ARGS);            \
    } while (0)
#define FLARE_DQ_NB(DD)                      \
    do {                                     \
        if (e.NB == 1) FLARE_DQ(DD, 1, 2);   \
        else FLARE_DQ(DD, 2, 2);             \
    } while (0)
    switch (s.d) {
        case 4: FLARE_DQ_NB(4); break;
        case 8: FLARE_DQ_NB(8); break;
        case 16: FLARE_DQ_NB(16); break;
        default:
            if (e.NB == 1) FLARE_DQ(32, 1, 2);
            else FLARE_DQ(32, 2, 1);
    }
#undef FLARE_DQ_NB
#undef FLARE_DQ
#undef FLARE_DQ_ARGS
    return check_launch();
}

// dK and dV of the backward.  One workgroup of 8 waves per (b,h) slice and block of token tiles;
// the operand images need dkdv_images KiB of LDS per latent tile.
// Workgroups per (b,h) (= dQ partial slots per (b,h) when it also forms dQ)
int mfma_dkdv_blocks(const flare_shape &s)
{
    const int BH = s.B * s.H;
    const int tiles = (s.N + 31) / 32;
    const int MT = lat_eff(s.M) / 32, waves = (mfma_dq_fused(s) && dkdv_pair(padded_dim(s.d), MT)) ? WV / 2 : WV;   // token tiles at a time
    const int most = BH <= 256 ? (256 + BH - 1) / BH : 4;   // one 8-wave workgroup per CU
    const int limit = min(4 * most, (tiles + waves - 1) / waves);
    // (setup: the operand images and the sum of the waves' dQ, 20 us beside 4.9 us a step at 256 latents and d = 16)
    return round_blocks(BH, 1, tiles, waves, 3 + 8 / MT, most, limit, kNever);
}

// The dK/dV kernel also forms the dQ partials (one pass over the scores for all three gradients).  At d <= 8
// it carries the lo term of Z in the upper half of its Z image (ZPACK in the kernel), like the token-statistics
// kernel that forms the delta it subtracts.  flare_shape.variant with FLARE_VARIANT_SEPARATE_DQ keeps the separate dQ
// kernel (tests, measurements), and so do few tokens beside chunks of seven or eight latent tiles at d = 32: each chunk is a launch
// whose workgroups sum the waves' dQ at its end (6 us), and one dQ kernel for all of them costs less where not every other
// pair of waves has a token tile (4 heads, 2644 tokens, 813 latents, backward 118 us fused, 103 apart; 72 heads, 306 tokens, 712
// latents 154 and 168; 16 heads and 2400 tokens or more 1.03 to 1.3 times as long apart).
bool mfma_dq_fused(const flare_shape &s)
{
    if (!mfma_supported(s)) return false;
    if (s.d == 32 && s.M > kLatChunk && lat_eff(s.M) > 192 && (long long)((s.N + 31) / 32) * s.B * s.H <= 2 * 256) return false;
    return (s.variant & FLARE_VARIANT_SEPARATE_DQ) == 0;
}

int mfma_dkdv(const flare_shape &s, const void *q, const void *k, const void *v, const void *dy, const float *z,
              const float *lse_enc, const float *lse_dec2, const float *delta,
              float ld_mul, void *dk, void *dv, float *acc32, float *dq_part, int m0, float scale,
              const MergeDz &merge_in, hipStream_t stream)
{
    // Both variants (one or two exponentials per score, whichever the plan names for a (b,h)) for the latent chunk
    // that starts at m0.  dq_part != NULL: also write the dQ partials (mfma_dq_fused(s) must hold), slot layout
    // [(b*h) * mfma_dkdv_blocks(s) + block][M][d]
    const int BH = s.B * s.H;
    const dim3 grid(mfma_dkdv_blocks(s), BH);
    const bool fuse = dq_part != nullptr;
    if (fuse && !mfma_dq_fused(s)) return FLARE_EUNSUPPORTED;
    const float c2 = scale * kLog2e;
    const int mend = min(s.M, m0 + lat_eff(s.M));
    int MT = lat_eff(s.M) / 32;
    const int pd = padded_dim(s.d);
    // dQ from this kernel at d = 16 with fewer tokens than latents: one more image, the lo term of Z (see the kernel)
    const bool zlo = fuse && s.d == 16 && s.N < s.M;
    // The forms that only few-token shapes and measurements take, and d = 4, exist for 1, 2, 4 and 8 tiles (and 7 at d = 32).
    if (zlo || s.d == 4 || (!fuse && !(s.d == 32 && MT == 7))) MT = MT <= 2 ? MT : MT <= 4 ? 4 : 8;
    if (fuse && dkdv_pair(s.d, MT)) MT += MT % 2;   // halved between two waves
    size_t lds = (size_t)MT * dkdv_images(s.d, fuse, zlo) * 1024 + (fuse ? WV * fused_wave_lds(pd, MT) * 2 : 0);
    MergeDz merge = merge_in;
    merge.lds = (unsigned)lds;
    if (merge.parts) lds += (size_t)s.M * (s.d + 1) * 4;
    const bf16_t *qq = (const bf16_t *)q, *kk = (const bf16_t *)k, *vv = (const bf16_t *)v, *gg = (const bf16_t *)dy;
    const bool f16 = s.dtype == FLARE_F16;
#define FLARE_DKDV_LAUNCH(KERN)                                                                                  \
    do {                                                                                                         \
        auto kern = KERN;                                                                                        \
        kern<<<grid, 64 * WV, lds, stream>>>(qq, kk, vv, gg, z, lse_enc, lse_dec2, delta, ld_mul, \
                                             (bf16_t *)dk, (bf16_t *)dv, acc32, dq_part, tok_stride(s), s.H,     \
                                             s.N, s.M, m0, mend, c2, scale, merge);                                    \
    } while (0)
    LaunchTimer t(KID_BWD_DKDV, stream);
#define FLARE_DKDV(DD, MTT, LO)                                                                 \
    do {                                                                                        \
        if (f16) FLARE_DKDV_LAUNCH((bwd_dkdv_planned_kernel<DD, MTT, LO, true>));               \
        else FLARE_DKDV_LAUNCH((bwd_dkdv_planned_kernel<DD, MTT, LO, false>));                  \
    } while (0)
#define FLARE_DKDV_POW2(DD, LO)                     \
    switch (MT) {                                   \
        case 1: FLARE_DKDV(DD, 1, LO); break;       \
        case 2: FLARE_DKDV(DD, 2, LO); break;       \
        case 4: FLARE_DKDV(DD, 4, LO); break;       \
        case 8: FLARE_DKDV(DD, 8, LO); break;       \
        default: return FLARE_EUNSUPPORTED;         \
    }
#define FLARE_DKDV_MT(DD, LO)                       \
    switch (MT) {                                   \
        case 3: FLARE_DKDV(DD, 3, LO); break;       \
        case 5: FLARE_DKDV(DD, 5, LO); break;       \
        case 6: FLARE_DKDV(DD, 6, LO); break;       \
        case 7: FLARE_DKDV(DD, 7, LO); break;       \
        default: FLARE_DKDV_POW2(DD, LO)            \
    }
    if (s.d == 4 && fuse) {
        FLARE_DKDV_POW2(4, true)
    } else if (s.d == 8 && fuse) {
        FLARE_DKDV_MT(8, true)
    } else if (s.d == 16 && fuse && zlo) {
#define FLARE_DKDV_Z(MTT)                                                                          \
    do {                                                                                           \
        if (f16) FLARE_DKDV_LAUNCH((bwd_dkdv_planned_kernel<16, MTT, true, true, true>));          \
        else FLARE_DKDV_LAUNCH((bwd_dkdv_planned_kernel<16, MTT, true, false, true>));             \
    } while (0)
        switch (MT) {
            case 1: FLARE_DKDV_Z(1); break;
            case 2: FLARE_DKDV_Z(2); break;
            case 4: FLARE_DKDV_Z(4); break;
            case 8: FLARE_DKDV_Z(8); break;
            default: return FLARE_EUNSUPPORTED;
        }
#undef FLARE_DKDV_Z
    } else if (s.d == 16 && fuse) {
        FLARE_DKDV_MT(16, true)
    } else if (s.d == 4) {
        FLARE_DKDV_POW2(4, false)
    } else if (s.d == 8) {
        FLARE_DKDV_POW2(8, false)
    } else if (s.d == 16) {
        FLARE_DKDV_POW2(16, false)
    } else if (fuse) {   // d = 32
        switch (MT) {
            case 1: FLARE_DKDV(32, 1, true); break;
            case 2: FLARE_DKDV(32, 2, true); break;
            case 3: FLARE_DKDV(32, 3, true); break;
            case 4: FLARE_DKDV(32, 4, true); break;
            case 6: FLARE_DKDV(32, 6, true); break;
            case 8: FLARE_DKDV(32, 8, true); break;
            default: return FLARE_EUNSUPPORTED;
        }
    } else if (MT == 7) {
        FLARE_DKDV(32, 7, false);
    } else {
        FLARE_DKDV_POW2(32, false)
    }
#undef FLARE_DKDV_MT
#undef FLARE_DKDV_POW2
#undef FLARE_DKDV
#undef FLARE_DKDV_LAUNCH
    return check_launch();
}

size_t mfma_dkdv_acc_bytes(const flare_shape &s)
{
    if (s.M <= kLatChunk) return 0;
    return ((size_t)s.B * s.H * s.N * s.d * 4 * 2 + 255) & ~(size_t)255;
}

// With few dZ slots the dK/dV kernel merges them.  Not with more than 256 latents, whose chunks are launches of
// their own, nor at d = 32 where the merged rows of more than 192 latents do not fit beside their images in LDS.
bool mfma_dz_inline(const flare_shape &s)
{
    return s.M <= kLatChunk && !(s.d == 32 && s.M > 192) && merge_inline(s, mfma_plan(s).parts);
}

// partial slots per (b,h) that mfma_dq_partial writes
int mfma_dq_parts(const flare_shape &s)
{
    const MfmaPlan p = mfma_plan(s);
    return p.enc.chunks * dq_geom(s).TG;
}

}  // namespace flare
