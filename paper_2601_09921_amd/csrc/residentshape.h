// What the two state-resident kernels (resident.hip, resident_split.hip) share: the shapes of the
// weight stream, the order of the per-layer vectors, and the attention of a feature group.
#pragma once
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace {

constexpr int FRAG = 512;          // bf16 values per fragment (1 KB)
constexpr int RCHUNK = 32;         // fragments per ring buffer
constexpr int RD = 128;            // d_model of the resident path
constexpr int RRT = RD / 16;       // 16-row C tiles of a d_model vector
constexpr int RKS = RD / 32;       // 32-deep k-steps of a d_model vector
constexpr int RMAXL = 4;           // layers whose vectors fit the LDS table

template <int MR>
struct RShape {
    static constexpr int F = MR * RD;
    static constexpr int CH = 64;                          // hidden units per feed-forward chunk
    static constexpr int NMLP = F / CH;
    static constexpr int QKV_FRAGS = 3 * 2 * RKS;          // Q, K, V of one 32-feature group
    static constexpr int W1_FRAGS = (CH / 16) * RKS, W2_FRAGS = RRT * (CH / 32);
    static constexpr int LAYER_CHUNKS = RKS + NMLP;
    static_assert(QKV_FRAGS + RRT == RCHUNK, "a Q/K/V group and its out-projection k-step fill one chunk");
    static_assert(W1_FRAGS + W2_FRAGS == RCHUNK, "a feed-forward chunk fills one ring buffer");
    static_assert(RKS % 2 == 0 && LAYER_CHUNKS % 2 == 0, "ring parity repeats every layer");
};

// Per-layer vectors, in the order the host writes them: [b_q b_k b_v | b_o g1 be1 b2 g2 be2 | b1].
template <int MR>
struct RVec {
    static constexpr int BQ = 0, BK = RD, BV = 2 * RD, BO = 3 * RD, G1 = 4 * RD, BE1 = 5 * RD, B2 = 6 * RD,
                         G2 = 7 * RD, BE2 = 8 * RD, B1 = 9 * RD;
    static constexpr int PER_LAYER = 9 * RD + MR * RD;
};

PWD_DEV bf16x4 to_b4(f32x4 v) {
    bf16x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (__bf16)v[i];
    return r;
}

// Softmax over the window's keys for NP independent (query block, head) pairs at once, so that
// their latencies overlap: scores s[p][kb] (keys 4g+i of key block kb as rows, this lane's
// query as the column), padding keys (index >= ntok, only ever in the last block) excluded.
// SHIFT: with the exact row maximum subtracted; otherwise exponentiated as they are. The
// probabilities, rounded to bf16, go to pb (the P^T operand); sum gets their column sum, taken
// on the matrix core from the same bf16 values (an A operand whose row 0 is all ones turns P^T
// into its column sums, in row 0 of the result), in every lane of the column, and inv 1 / sum.
template <bool SHIFT, int NP, int TB>
PWD_DEV void softmax_cols(f32x4 (&s)[NP][TB], bf16x4 (&pb)[NP][TB], float (&sum)[NP], float (&inv)[NP], int ntok,
                          int g, bf16x4 ones) {
    if (ntok < TB * 16) {   // wavefront-uniform: the last block holds padding keys
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((TB - 1) * 16 + 4 * g + i >= ntok) s[p][TB - 1][i] = -INFINITY;
    }
    float mx[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) mx[p] = 0.f;
    if constexpr (SHIFT) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            mx[p] = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < TB; ++kb)
                mx[p] = fmaxf(mx[p], fmaxf(fmaxf(s[p][kb][0], s[p][kb][1]), fmaxf(s[p][kb][2], s[p][kb][3])));
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) mx[p] = group_max(mx[p]);
    }
    f32x4 ls[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        ls[p] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < TB; ++kb) {
            f32x4 e;
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(SHIFT ? s[p][kb][i] - mx[p] : s[p][kb][i]);
            pb[p][kb] = to_b4(e);
            ls[p] = mfma16x16x16(ones, pb[p][kb], ls[p]);
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        sum[p] = row0_broadcast(ls[p][0]);
        inv[p] = __builtin_amdgcn_rcpf(sum[p]);
    }
}

// True (wavefront-uniform) when every column sum lies in [1e-30, 2^126] and every output value
// is finite (x * 0 is 0 for finite x and NaN otherwise): the unshifted softmax is then the exact
// one up to rounding. Otherwise the caller recomputes with the row maximum subtracted.
template <int NP>
PWD_DEV bool in_range(const float (&sum)[NP], const f32x4 (&o)[NP]) {
    bool ok = true;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        float chk = sum[p];
#pragma unroll
        for (int i = 0; i < 4; ++i) chk = fmaf(o[p][i], 0.f, chk);
        ok = ok && chk >= 1e-30f && chk <= 0x1p126f;
    }
    return __builtin_amdgcn_ballot_w64(!ok) == 0;
}

// Attention of a 32-feature group's heads (two of 16 features or one of 32) from its Q, K and V
// accumulators over the window's TB blocks: y[qb] = O^T of query block qb as a B fragment.
template <int TB, int DH>
PWD_DEV void attend_group(const f32x4 (&q)[2][TB], const f32x4 (&k)[2][TB], const f32x4 (&v)[2][TB], bf16x8 (&y)[TB],
          float qscale, int ntok, int g, bf16x4 ones) {
    bf16x4 vt[2][TB];   // V^T A operands per 16-feature tile and key block
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int b = 0; b < TB; ++b) vt[hh][b] = to_b4(v[hh][b]);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if constexpr (DH == 16) {   // two heads per group: features 16 hh .. 16 hh + 15
        constexpr int NP = 2 * TB;   // pair p = query block p / 2, head p % 2
        bf16x4 q4[2][TB], k4[2][TB];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                q4[hh][b] = to_b4(q[hh][b] * qscale);
                k4[hh][b] = to_b4(k[hh][b]);
            }
        f32x4 o[NP];
        float inv[NP];
        auto attend = [&](auto shift) {
            f32x4 s[NP][TB];
            bf16x4 pb[NP][TB];
            float sum[NP];
#pragma unroll
            for (int pp = 0; pp < NP; ++pp)
#pragma unroll
                for (int kb = 0; kb < TB; ++kb) s[pp][kb] = mfma16x16x16(k4[pp % 2][kb], q4[pp % 2][pp / 2], zero);
            softmax_cols<decltype(shift)::value, NP, TB>(s, pb, sum, inv, ntok, g, ones);
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) {
                o[pp] = zero;
#pragma unroll
                for (int kb = 0; kb < TB; ++kb) o[pp] = mfma16x16x16(vt[pp % 2][kb], pb[pp][kb], o[pp]);
            }
            return in_range<NP>(sum, o);
        };
        if (!attend(std::false_type{})) attend(std::true_type{});
#pragma unroll
        for (int qb = 0; qb < TB; ++qb) y[qb] = pack_b(o[2 * qb] * inv[2 * qb], o[2 * qb + 1] * inv[2 * qb + 1]);
    } else {   // one head of 32 features
        bf16x8 qf[TB], kf[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            qf[b] = pack_b(q[0][b] * qscale, q[1][b] * qscale);
            kf[b] = pack_b(k[0][b], k[1][b]);
        }
        f32x4 o[TB][2];
        float inv[TB];
        auto attend = [&](auto shift) {
            f32x4 s[TB][TB];
            bf16x4 pb[TB][TB];
            float sum[TB];
#pragma unroll
            for (int qb = 0; qb < TB; ++qb)
#pragma unroll
                for (int kb = 0; kb < TB; ++kb) s[qb][kb] = mfma16x16x32(kf[kb], qf[qb], zero);
            softmax_cols<decltype(shift)::value, TB, TB>(s, pb, sum, inv, ntok, g, ones);
#pragma unroll
            for (int qb = 0; qb < TB; ++qb)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    o[qb][hh] = zero;
#pragma unroll
                    for (int kb = 0; kb < TB; ++kb) o[qb][hh] = mfma16x16x16(vt[hh][kb], pb[qb][kb], o[qb][hh]);
                }
            // both halves of each query block's output against its sum
            float sum2[2 * TB];
            f32x4 o2[2 * TB];
#pragma unroll
            for (int qb = 0; qb < TB; ++qb)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    sum2[2 * qb + hh] = sum[qb];
                    o2[2 * qb + hh] = o[qb][hh];
                }
            return in_range<2 * TB>(sum2, o2);
        };
        if (!attend(std::false_type{})) attend(std::true_type{});
#pragma unroll
        for (int qb = 0; qb < TB; ++qb) y[qb] = pack_b(o[qb][0] * inv[qb], o[qb][1] * inv[qb]);
    }
}

}  // namespace
