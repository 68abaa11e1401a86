// What the two token-local kernels (tok.hip, wide.hip) share: the shapes of the weight streams, the
// order of the vector tables, and the event lookup and fold of the embedding.
#pragma once
#include "common.h"
#include "kernels.h"

namespace {

constexpr int FRAG = 512;       // bf16 values per fragment (1 KB)

template <int D, int NW, int MR>
struct Shape {
    static constexpr int CHUNK = 32;                  // weight fragments per LDS chunk
    static constexpr int RT = D / 16;                 // 16-row C tiles of a D-vector
    static constexpr int KS = D / 32;                 // 32-deep k-steps of a D-vector
    static constexpr int F = MR * D;                  // feed-forward width (MR = 4 or 5)
    static constexpr int CH = 8192 / D;               // hidden units per feed-forward chunk
    static constexpr int NMLP = F / CH;               // feed-forward sub-chunks (32 fragments each)
    static constexpr int MLP_PER = CHUNK / 32;        // feed-forward sub-chunks per LDS chunk
    static constexpr int MLP_CHUNKS = NMLP / MLP_PER;
    static constexpr int WO_CHUNKS = RT * KS / CHUNK;
    static constexpr int QKV_CHUNKS = (3 * D / 16) * KS / CHUNK;
    static constexpr int OG_PER_CHUNK = CHUNK / (2 * KS);
    static constexpr int POST_CHUNKS = WO_CHUNKS + MLP_CHUNKS;
    static_assert((CH / 16) * KS + RT * (CH / 32) == 32, "32 fragments per feed-forward sub-chunk");
    // MXFP8 (TOK_MX): 8-bit fragments of 16 rows x 128 k (2 KB, two 1 KB halves = two reads).
    // A feed-forward chunk holds the CH hidden units' W1 fragments (hidden row tile, k-step)
    // followed by their bf16 W2 fragments, a Q/K/V chunk 12 fragments (output group, k-step,
    // row tile); slot MX_SCALE_SLOT holds the chunk's weight scales, lane-major, byte j of a
    // lane for 8-bit fragment j; the other slots are unused.
    static constexpr int KS8 = D / 128;
    static constexpr int MX_SCALE_SLOT = 24;
    static constexpr int MX_NW1 = (CH / 16) * KS8;
    static constexpr int MX_FFN_READS = 2 * MX_NW1 + RT * (CH / 32);
    static constexpr int MX_QKV_FRAGS = 12;
    static constexpr int MX_OPC = MX_QKV_FRAGS / (2 * KS8);   // output groups per Q/K/V chunk
    static constexpr int MX_QKV_READS = 2 * MX_QKV_FRAGS;
    static constexpr int MX_QKV_CHUNKS = (3 * D / 32) / MX_OPC;
    static_assert(MX_FFN_READS == MX_SCALE_SLOT && MX_QKV_READS == MX_SCALE_SLOT, "data ahead of the scales");
    static_assert((3 * D / 32) % MX_OPC == 0 && MX_NW1 <= 4 && MLP_PER == 1, "MXFP8 chunk layout");
    static_assert(NMLP % MLP_PER == 0, "whole feed-forward chunks");
    static_assert(RT * KS % CHUNK == 0 && (3 * D / 16) * KS % CHUNK == 0, "whole chunks");
};

PWD_DEV u16x4 to_bf16x4(f32x4 v) {
    u16x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_bit_cast(uint16_t, (__bf16)v[i]);
    return r;
}

PWD_DEV f32x4 relu4(f32x4 v) {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = v[i] > 0.f ? v[i] : 0.f;
    return r;
}

// LDS of one workgroup (two per CU): the weight ring (two 32-fragment buffers) + vectors.
constexpr int LDS_BUDGET = 80 * 1024, RING_BYTES = 2 * 32 * FRAG * 2;

// b_v is stored with each value four times (the bias of a V tile is one column value per
// lane, loaded as the f32x4 an accumulator starts from) where that fits in LDS, else once.
constexpr int bv_rep(int D, int F) { return (12 * D + F) * 4 + RING_BYTES <= LDS_BUDGET ? 4 : 1; }

// Per-launch vectors staged in LDS once: [bo g1 be1 b2 g2 be2 | b1 (F) | b_q b_k | b_v].
template <int D, int F>
struct Vecs {
    static constexpr int BO = 0, G1 = D, BE1 = 2 * D, B2 = 3 * D, G2 = 4 * D, BE2 = 5 * D;
    static constexpr int REP = bv_rep(D, F);
    static constexpr int B1 = 6 * D, BQKV = 6 * D + F, BV = BQKV + 2 * D, QKV_VECS = (2 + REP) * D;
    static constexpr int SIZE = BQKV + QKV_VECS;
    static_assert(SIZE * 4 + RING_BYTES <= LDS_BUDGET, "vector table fits");
};

// Detection event (0 or 1) of round p.t for column `col`'s token of token block tb, and with RES
// the token's row of the embedder block's table; 0 and row 0 for padding.
template <bool RES>
PWD_DEV void token_event(const TokParams& p, int64_t tb, int col, float& ev, int& row) {
    const int64_t w = tb / p.nbw;
    const int s = (int)(tb - w * p.nbw) * 16 + col;   // token
    ev = 0.f;
    row = 0;
    const int st = s < p.ntok ? (p.tok_stab ? p.tok_stab[s] : s) : -1;   // its stabilizer
    if (w < p.in.nwin) {
        const uint32_t* m = p.in.meas + w * (int64_t)(p.in.W + 1) * p.in.words;
        const int type = p.in.types[w];
        auto bit = [&](int q) -> uint32_t {   // event of stabilizer q in round t
            const uint32_t word = event_word(m, p.in.words, p.t, q >> 5, type, p.in.b_left, p.in.d);
            return (word >> (q & 31)) & 1u;
        };
        if (st >= 0) ev = (float)bit(st);
        if constexpr (RES) {
            if (s < p.ntok) {
                const int* nb = p.emb_nb + (size_t)s * 8;
                uint32_t pat = 0u;
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    const int q = nb[j];
                    if (q >= 0) pat |= bit(q) << j;
                }
                row = nb[5] * 32 + (int)pat;
            }
        }
    }
}

// Embedding and fold of one value: X = kappa (E w_e + b_e + PE + X), the embedding 0 on padding.
PWD_DEV float fold(bool real, float e, float we, float s0, float prev, float kappa) {
    const float emb = real ? e * we + s0 : 0.f;
    return kappa * (emb + prev);
}

}  // namespace
