// fp32 decoder for small windows: one workgroup runs one window through every round,
// layer and the readout with its whole state on chip (Algorithm 1, inference branch, or the
// recurrent branch's readout after each of the last rounds; App. A model). Used for the fp32
// configurations (d_model <= 64, about d <= 5), where a window is a few kilobytes and the batch
// is small, so one launch per decode is the point.
//
// Matrix products run on the matrix core in fp32, v_mfma_f32_4x4x1_16b: 16 blocks of 4 rows x 4
// columns with one k each, block b's rows broadcast over a group of blocks (CBSZ / ABID). The
// four rows are tokens and the 64 lanes output features, so a weight register is a row of W as
// it lies in memory (64 features at one k; 32 and 16 at d_model 32 and 16, whose lane groups
// take 2 and 4 token quads), one activation register holds 4 tokens x 16 (8, 4) k values, and a
// window of 8 or 24 tokens wastes no columns -- a 16-column tile would compute half of its
// columns for nothing at 8 tokens. What bounds it: the weights, which every workgroup pulls
// from L2 once per layer and round (48 D^2 bytes, at 64 bytes per cycle and CU as long as the
// matrix core needs for 8 tokens), and the seven dependent phases of a layer. So each matrix's
// weights are split over the wavefronts by output columns or by k, loaded straight into the
// registers of the wavefront that multiplies them (no LDS pass) and refilled right after use,
// two phases to a layer ahead. Products split by k leave one partial sum per
// wavefront in LDS, which the phase that reads them adds up.
// Measured: d 3, d_model 64, 64 windows of 6 rounds 61 us; d 5, d_model 32, 1000 windows of 15
// rounds 437 us (with FMA loops over LDS operands and one weight load per FMA: 636 and 5167 us).
// With the refills after a product instead of between its instructions, 66 us at d 3.
//
// Every output element is summed in a fixed order, so results do not depend on the batch.
#include "common.h"
#include "kernels.h"
#include "pipeline.h"

#include <cstddef>

namespace {

// Compile-time shape: d_model D, feed-forward width MR * D, NT token tiles.
template <int D, int MR, int NT>
struct F32Shape {
    static constexpr int F = MR * D;
    static constexpr int WAVES = D == 64 ? 8 : 4, THREADS = WAVES * 64;
    static constexpr int KP = WAVES / 4;             // k halves of the Q/K/V and first feed-forward products
    static constexpr int TQ = 256 / D;               // tokens per MFMA (4 per group of D lanes)
    static constexpr int KA = D / 4;                 // k values per activation register
    static constexpr int CBSZ = D == 64 ? 4 : D == 32 ? 3 : 2;
    static constexpr int NP = NT * TQ;               // token rows held in LDS
    static constexpr int NKB = (NP + 15) / 16;       // 16-key blocks of the attention
    static constexpr int TPP = THREADS / D;          // tokens per pass of the elementwise phases
    static constexpr int NE = (NP + TPP - 1) / TPP;  // elements of the state each thread owns
    static constexpr int KQ = D / KP, KO = D / WAVES, KW2 = F / WAVES, KR = 4 * D / WAVES;   // k per wavefront
    // LDS row strides: the activation read (TQ rows x KA consecutive) and the attention's operand
    // reads (16 rows x 4, 4 rows 4 apart x 16) fall on distinct banks
    static constexpr int SX = D + KA, S3 = 3 * D + 4, SF = F + KA;
    static constexpr int cmax(int a, int b) { return a > b ? a : b; }
    // regions: the state; Q/K/V partials, then the partials of products split by k; attention
    // output, then hidden units
    static constexpr int R1 = cmax(KP * NP * S3, WAVES * NP * D), R2 = cmax(KP * NP * SF, NP * SX);
    // readout: position tiles of the largest distance with this many token rows, one partial
    // result per wavefront over R1 and R2
    static constexpr int PMAX = NP <= 16 ? 9 : NP <= 32 ? 25 : D == 16 ? 49 : 25;
    static constexpr int PT = (PMAX + TQ - 1) / TQ;
    static constexpr int R12 = cmax(R1 + R2, WAVES * PT * TQ * D);
    static constexpr int VEC = 9 * D + F;            // vectors of a layer
    static constexpr int RTAB = 4 * PT * TQ, CTAB = 27 * NP;   // gather tables (see the kernel)
    static constexpr size_t smem(int L, bool conv) {
        return sizeof(float) * ((size_t)NP * SX + R12 + WAVES + (size_t)L * VEC + RTAB + (conv ? CTAB : 0));
    }
};

// Per layer: bq bk bv bo g1 be1 b2 g2 be2 b1.
template <int D>
struct F32Vec {
    static constexpr int BQKV = 0, BO = 3 * D, G1 = 4 * D, BE1 = 5 * D, B2 = 6 * D, G2 = 7 * D, BE2 = 8 * D, B1 = 9 * D;
};

template <int CTRL>
PWD_DEV float dpp(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// Sum over aligned groups of D lanes (16, 32 or 64), in every lane of the group: within a row of
// 16 with lane permutations of the vector ALU (xor 1, xor 2, half mirror, mirror), across rows
// with the lane swaps.
template <int D>
PWD_DEV float lane_sum(float v) {
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    v += dpp<0x140>(v);
    float o;
    if constexpr (D >= 32) {
        const float a = swap16(v, o);
        v = a + o;
    }
    if constexpr (D >= 64) {
        const float a = swap32(v, o);
        v = a + o;
    }
    return v;
}

// v itself, as a value the compiler does not move out of loops: the many addresses that derive
// from it are computed where they are used instead of being kept in registers for the whole
// kernel (which would spill the weights).
PWD_DEV int here(int v) { return __builtin_amdgcn_update_dpp(0, v, 0xE4, 0xf, 0xf, true); }

PWD_DEV f32x4 mfma16x16x4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// the weights at base + off replace w (nothing without a base)
PWD_DEV void refill(f32x4& w, const float* base, int off) {
    __builtin_amdgcn_sched_barrier(0);   // after the last use of what it replaces
    w = ld4(base + off);
}
PWD_DEV void refill(f32x4&, std::nullptr_t, int) {}

// Wavefronts per SIMD that the registers are limited for (128, 168 or 256), at d_model 32 and 2 layers,
// 4096 windows (and 64) with four / three / two, us:
//     tokens, F/D   four          three         two
//     8, 5          326 (55)      347 (49)      345 (48)
//     16, 4         397 (59)      421 (55)      420 (56)
//     16, 5         467 (75)      490 (70)      483 (64)
//     24, 4         1090 (153)    1123 (136)    1086 (128)
//     24, 5         1431 (204)    1291 (161)    1227 (144)
//     36, 4         2206 (249)    1704 (203)    2011 (197)
//     36, 5         3110 (294)    2415 (246)    2312 (231)
// (8, 4 fits 128 registers.) Four cost spills, 40 registers at 24 tokens and F = 4 D, but let four
// workgroups share a CU, which is a whole batch of 1000 windows at once: 437 against 477 us with three for
// the 15 rounds above. At 24 tokens and F = 5 D, and from 25 tokens on, the spills cost more than that. At
// F = 5 D two wavefronts give the better code (24 tokens: 163 registers, so three still fit); at 36
// tokens and F = 4 D they leave too few workgroups. At d_model 16 the choice changes less than 3 %, but
// for 64 tokens and F = 5 D (1617, 1536, 1508 us).
template <int D, int MR, int NT>
constexpr int f32_waves() { return D == 64 ? 2 : NT + MR <= 7 ? 4 : MR == 4 ? 3 : 2; }

template <int D, int MR, int NT>
__global__ __launch_bounds__((F32Shape<D, MR, NT>::THREADS), (f32_waves<D, MR, NT>())) void f32_window_kernel(F32Params p) {
    using S = F32Shape<D, MR, NT>;
    using V = F32Vec<D>;
    constexpr int WAVES = S::WAVES, KP = S::KP, TQ = S::TQ, KA = S::KA, NP = S::NP, NKB = S::NKB;
    constexpr int NE = S::NE, TPP = S::TPP, SX = S::SX, S3 = S::S3, SF = S::SF;
    const int win = blockIdx.x;
    const int N = p.ntok, H = p.H, dh = D / H, d = p.in.d;
    extern __shared__ __align__(16) float sm[];
    float* X = sm;                      // [NP][SX] state / residual stream
    float* QP = X + NP * SX;            // R1: [KP][NP][S3] Q, K, V (k partials, without biases) ...
    float* WP = QP;                     // ... or [WAVES][NP][D] k partials of a product
    float* HP = QP + S::R1;             // R2: [KP][NP][SF] hidden units before bias and ReLU ...
    float* AO = HP;                     // ... or [NP][SX] attention output
    float* red = QP + S::R12;           // [WAVES]
    float* vec = red + WAVES;           // [L][VEC]
    // offsets in X of the gathered products' rows, -1 where there is none: the readout's by (tap,
    // position), a convolution's by (unit, tap, token)
    int* rtab = reinterpret_cast<int*>(vec + p.L * S::VEC);   // [4][PT * TQ]
    int* ctab = rtab + S::RTAB;                               // [3][9][NP]

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // products split by columns may leave wavefronts without work; which ones rotates with the
    // window, so that the workgroups of a CU do not all leave the same SIMD idle
    const int role = (wave + (D == 64 ? 0 : win)) & (WAVES - 1);
    // a lane's part of the products, derived anew in each phase
    struct Lane {
        int lane, col;     // its column of a column group
        int trow, tk;      // token and k of its value of an activation register
        int c4;            // first token of its result registers
        __device__ Lane() {
            lane = here((int)threadIdx.x & 63);
            col = lane % D;
            trow = 4 * (lane / D) + (lane & 3);
            tk = col >> 2;
            c4 = 4 * (lane / D);
        }
    };

    // element (token n0 + e TPP, feature f) of the state, owned by this thread in registers too
    struct Own {
        int f, n0;
        __device__ Own() {
            const int i = here((int)threadIdx.x);
            f = i % D;
            n0 = i / D;
        }
    };

    // ---- weights: [column group][k / 4][D columns][4] per matrix; per layer Wqkv (3 groups),
    // Wo, W1 (MR groups), W2
    constexpr int WQKV = 0, WO = 3 * D * D, W1 = 4 * D * D, W2 = W1 + MR * D * D, LAYER = W2 + MR * D * D;
    // this wavefront's columns and k range of each product
    const bool has_q = role < 3 * KP;   // without: the loads repeat another's, nothing is computed
    const int cgq = role % 3, kpq = has_q ? role / 3 : 0;
    const int cg1 = role % 4, kp1 = role / 4;            // the fifth group of MR = 5 is shared out below
    auto load_w = [&](auto& w, const float* base) {
        constexpr int n = sizeof(w) / sizeof(f32x4);
        const int col = Lane().col;
#pragma unroll
        for (int j = 0; j < n; ++j) w[j] = ld4(base + (j * D + col) * 4);
    };
    // wa: Wqkv, then (refilled while the attention runs) W1, then the next layer's Wqkv
    f32x4 wa[S::KQ / 4], wo[S::KO / 4], w2[S::KW2 / 4];
    // where each product's weights of a layer start (first group of four k of this wavefront)
    auto src_wq = [&](const float* w) { return w + WQKV + cgq * D * D + kpq * S::KQ * D; };
    auto src_wo = [&](const float* w) { return w + WO + wave * S::KO * D; };
    auto src_w1 = [&](const float* w) { return w + W1 + cg1 * D * D + kp1 * S::KQ * D; };
    auto src_w2 = [&](const float* w) { return w + W2 + wave * S::KW2 * D; };
    load_w(wa, src_wq(p.stream));
    load_w(wo, src_wo(p.stream));
    load_w(w2, src_w2(p.stream));

    // acc[t] += sum over KW k of a(token row of tile t, k) w[k], even and odd k in sums of their own
    // (shorter dependent chains, and half the accumulated rounding); a(t, row, k) reads one
    // activation. With `next`, each group of four k is reloaded from there right after its last
    // use: spread between the products like this, the loads' issue (16 cycles each on the CU's
    // one path to L1) overlaps them instead of following them.
    auto gemm = [&](auto& acc, auto& w, const auto& a, auto next) {
        const Lane ln;
        constexpr int KW = (int)(sizeof(w) / sizeof(f32x4)) * 4, T = (int)(sizeof(acc) / sizeof(f32x4));
        f32x4 odd[T];
#pragma unroll
        for (int t = 0; t < T; ++t) odd[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        static_for<(KW + KA - 1) / KA>([&](auto kg) {
            constexpr int K0 = decltype(kg)::value * KA;
            float av[T];
#pragma unroll
            for (int t = 0; t < T; ++t) av[t] = a(t, t * TQ + ln.trow, K0 + ln.tk);
            static_for<(KW - K0 < KA ? KW - K0 : KA)>([&](auto kk) {
                constexpr int K = K0 + decltype(kk)::value;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    f32x4& s = K % 2 ? odd[t] : acc[t];
                    s = __builtin_amdgcn_mfma_f32_4x4x1f32(av[t], w[K / 4][K % 4], s, S::CBSZ, decltype(kk)::value, 0);
                }
                if constexpr (K % 4 == 3) refill(w[K / 4], next, (K / 4 * D + ln.col) * 4);
            });
        });
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] += odd[t];
    };
    // results to rows of `out` (stride so), column c0 of this lane's group
    auto store = [&](float* out, int so, const auto& acc) {
        const Lane ln;
        constexpr int T = (int)(sizeof(acc) / sizeof(f32x4));
        float* dst = out + ln.c4 * so + ln.col;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[(t * TQ + i) * so] = acc[t][i];
    };
    auto clear = [&](auto& acc) {
        for (auto& v : acc) v = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // accumulators start at the column's bias in the wavefront with the first k range, else at 0
    auto start = [&](auto& acc, const float* b, int kp) {
        const float v = kp == 0 ? b[Lane().col] : 0.f;
        for (auto& a : acc) a = f32x4{v, v, v, v};
    };

    for (int i = tid; i < p.L * S::VEC; i += S::THREADS) vec[i] = p.vecs[i];
    // the state's rows past N, which the products read, stay zero: their results, in rows past N
    // again, are never read as a token's
    for (int i = tid; i < NP * SX + S::R12; i += S::THREADS) X[i] = 0.f;
    for (int i = tid; i < S::RTAB; i += S::THREADS) {
        const int tap = i / (S::PT * TQ), pos = i % (S::PT * TQ);
        int tok = -1;
        if (pos < d * d) tok = p.cell_token[(pos / d + (tap >> 1)) * (d + 1) + pos % d + (tap & 1)];
        rtab[i] = tok >= 0 ? tok * SX : -1;
    }
    if (p.conv_w)
        for (int i = tid; i < S::CTAB; i += S::THREADS) {
            const int side = d + 1, j = i / (9 * NP), tap = i / NP % 9, n = i % NP;
            const int r = n / side + p.dil[j] * (tap / 3 - 1), c = n % side + p.dil[j] * (tap % 3 - 1);
            ctab[i] = n < N && r >= 0 && r < side && c >= 0 && c < side ? (r * side + c) * SX : -1;
        }
    const int type = p.in.types[win];
    const uint32_t* meas = p.in.meas + (int64_t)win * (p.in.W + 1) * p.in.words;
    const Own own0;
    const float we = p.we[own0.f];
    float x[NE], s0[NE];
    int st[NE];                          // the element's stabilizer, or -1
    uint32_t m_prev[NE], m_cur[NE];      // its measurement words of rows t and t + 1
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int n = own0.n0 + e * TPP;
        x[e] = 0.f;
        st[e] = -1;
        s0[e] = 0.f;
        if (n < N) {
            st[e] = p.tok_stab ? p.tok_stab[n] : n;
            s0[e] = p.S0[n * D + own0.f];
        }
        const int wd = st[e] >= 0 ? st[e] >> 5 : 0;
        m_prev[e] = meas[wd];
        m_cur[e] = meas[p.in.words + wd];
    }
    __syncthreads();   // the cleared state before it is written

    // readout (App. A.3) of the state in X into output slot k: 2x2 valid convolution + ReLU,
    // mean over columns, linear; positions are the rows of the product, the four taps its k,
    // split over the wavefronts; one fixed-order reduction over the workgroup
    auto readout = [&](int k) {
        const int k0 = wave * S::KR, tap = k0 / D;       // a wavefront's k lie within one tap
        const Lane ln;
        f32x4 acc[S::PT];
        int src[S::PT];
#pragma unroll
        for (int t = 0; t < S::PT; ++t) src[t] = rtab[tap * S::PT * TQ + t * TQ + ln.trow];
        clear(acc);
#pragma unroll 1
        for (int kg = 0; kg < S::KR; kg += KA) {
            f32x4 wr[KA / 4];
            load_w(wr, p.wc + (k0 + kg) * D);
            gemm(acc, wr, [&](int t, int, int kk) { return src[t] >= 0 ? X[src[t] + k0 % D + kg + kk] : 0.f; }, nullptr);
        }
        store(QP + wave * S::PT * TQ * D, D, acc);
        __syncthreads();
        float part = 0.f;
        for (int idx = here(tid); idx < d * D; idx += S::THREADS) {
            const int i = idx / D, o = idx % D;
            const float bc = p.bc[o];
            float pool = 0.f;
            for (int j = 0; j < d; ++j) {
                float v = bc;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) v += QP[(w * S::PT * TQ + i * d + j) * D + o];
                pool += fmaxf(v, 0.f);
            }
            part = fmaf(p.wo[idx], pool / (float)d, part);
        }
        part = lane_sum<64>(part);
        if ((tid & 63) == 0) red[wave] = part;
        __syncthreads();
        if (tid == 0) {
            float tot = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) tot += red[w];
            const int64_t o = (int64_t)win * p.readouts + k;
            if (type > WIN_FINAL) {
                p.logits[o] = __builtin_nanf("");
                p.bits[o] = 0;
                atomicOr(p.err, 1);
            } else {
                const float logit = tot + p.bo + p.beta[type];
                p.logits[o] = logit;
                p.bits[o] = logit > 0.f ? 1 : 0;
            }
        }
        __syncthreads();   // red and the partials are reused
    };

    // LayerNorm of x + b + the WAVES partials in WP, over the D lanes that share a token (two
    // passes, biased variance); the result stays in x
    auto add_norm = [&](const float* b, const float* g, const float* be) {
        const Own o;
        const int f = o.f, n0 = o.n0;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int n = n0 + e * TPP;
            if (n < N) {   // wavefront-uniform: a wavefront's 64 / D tokens divide N
                float y = b[f];
#pragma unroll
                for (int w = 0; w < WAVES; ++w) y += WP[(w * NP + n) * D + f];
                y += x[e];
                const float c = y - lane_sum<D>(y) * (1.f / D);
                const float rstd = rsqrtf(lane_sum<D>(c * c) * (1.f / D) + p.eps);
                x[e] = c * rstd * g[f] + be[f];
            }
        }
    };
    auto publish = [&]() {
        const Own o;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (o.n0 + e * TPP < N) X[(o.n0 + e * TPP) * SX + o.f] = x[e];
    };

    // one (head, 16-query block): S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_16x16x4: a result
    // register i of S^T (keys 4 g + i) is the operand of the product over those four keys. Keys from N
    // on get score -inf and V = 0, so nothing that LDS holds there counts; rows from NP on (the last
    // block's, where NP is no multiple of 16) belong to other values, which other wavefronts may be
    // writing, and are not read: block row 0 stands in for them.
    auto attend = [&](int h, int qb) {
        const int lane = here(tid & 63), g = lane >> 4, c16 = lane & 15;
        auto inside = [&](int kb, int r) { return (kb + 1) * 16 <= NP || kb * 16 + r < NP ? r : 0; };
        auto at = [&](int row, int cc) {   // Q, K or V element: its k partials
            float v = QP[row * S3 + cc];
            if constexpr (KP == 2) v += QP[(NP + row) * S3 + cc];
            return v;
        };
        const int q = qb * 16 + c16, qrow = NP % 16 == 0 || q < NP ? q : 0;
        f32x4 s[NKB];
        clear(s);
        // STEPS k-steps of four features from feature cc: their operands are read ahead of the products
        auto scores = [&](auto steps, int cc) {
            constexpr int STEPS = decltype(steps)::value;
            float a[STEPS][NKB], b[STEPS];
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                b[k] = at(qrow, cc + 4 * k);
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) a[k][kb] = at(kb * 16 + inside(kb, c16), D + cc + 4 * k);
            }
#pragma unroll
            for (int k = 0; k < STEPS; ++k)
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) s[kb] = mfma16x16x4(a[k][kb], b[k], s[kb]);
        };
        if (dh % 16 == 0)
            for (int c0 = 0; c0 < dh; c0 += 16) scores(std::integral_constant<int, 4>{}, h * dh + c0 + g);
        else if (dh == 8) scores(std::integral_constant<int, 2>{}, h * dh + g);
        else scores(std::integral_constant<int, 1>{}, h * dh + g);   // 4
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[kb][i] = kb * 16 + 4 * g + i < N ? s[kb][i] * p.scale : -INFINITY;
                mx = fmaxf(mx, s[kb][i]);
            }
        mx = group_max(mx);
        float sum = 0.f;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[kb][i] = expf(s[kb][i] - mx);
                sum += s[kb][i];
            }
        const float inv = 1.f / group_sum(sum);
        for (int r0 = 0; r0 < dh; r0 += 16) {
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
            const int row = r0 + c16 < dh ? r0 + c16 : 0;   // rows past the head's features: unused
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // N > NP - TQ: only the last blocks can hold rows past it
                    float v = at(kb * 16 + inside(kb, 4 * g) + i, 2 * D + h * dh + row);
                    if ((kb + 1) * 16 > NP - TQ) v = kb * 16 + 4 * g + i < N ? v : 0.f;
                    o = mfma16x16x4(v, s[kb][i], o);
                }
            if (q < N && r0 + 4 * g < dh) *reinterpret_cast<f32x4*>(AO + q * SX + h * dh + r0 + 4 * g) = o * inv;
        }
    };

    for (int t = 0; t < p.in.W; ++t) {
        const Own o;
        const int f = o.f, n0 = o.n0;
        // embedding + fold: X = kappa (E w_e + b_e + PE + X), X = 0 before round 0; with the
        // embedder's residual block, plus its output looked up by the events of the five cells
        // around the token's cell and the cell's position class
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int n = n0 + e * TPP;
            if (n < N) {
                uint32_t bit = 0u;
                if (type <= WIN_FINAL && st[e] >= 0)
                    bit = (event_from(m_prev[e], m_cur[e], t, type, p.in.b_left, d) >> (st[e] & 31)) & 1u;
                float s = fmaf((float)bit, we, s0[e]);
                if (p.emb_tab) {
                    const int* nb = p.emb_nb + n * 8;
                    uint32_t pat = 0u;
                    if (type <= WIN_FINAL)
#pragma unroll
                        for (int j = 0; j < 5; ++j)
                            if (nb[j] >= 0)
                                pat |= ((event_word(meas, p.in.words, t, nb[j] >> 5, type, p.in.b_left, d) >> (nb[j] & 31)) & 1u) << j;
                    s += p.emb_tab[(size_t)(nb[5] * 32 + (int)pat) * D + f];
                }
                x[e] = p.kappa * (s + x[e]);
            }
            m_prev[e] = m_cur[e];
            if (t + 2 <= p.in.W) m_cur[e] = meas[(t + 2) * p.in.words + (st[e] >= 0 ? st[e] >> 5 : 0)];
        }
        publish();
        __syncthreads();
        for (int l = 0; l < p.L; ++l) {
            const float* vl = vec + l * S::VEC;
            const float* wl = p.stream + (size_t)l * LAYER;
            const float* wn = p.stream + (size_t)(l + 1 < p.L ? l + 1 : 0) * LAYER;   // the next layer's
            f32x4 acc[NT];
            if (has_q) {
                start(acc, vl + V::BQKV + cgq * D, kpq);
                gemm(acc, wa, [&](int, int r, int k) { return X[r * SX + kpq * S::KQ + k]; }, src_w1(wl));
                store(QP + kpq * NP * S3 + cgq * D, S3, acc);
            } else {
                load_w(wa, src_w1(wl));
            }
            __syncthreads();
            for (int task = wave; task < H * NKB; task += WAVES) attend(task / NKB, task % NKB);
            __syncthreads();
            clear(acc);
            gemm(acc, wo, [&](int, int r, int k) { return AO[r * SX + wave * S::KO + k]; }, src_wo(wn));
            store(WP + wave * NP * D, D, acc);
            __syncthreads();
            add_norm(vl + V::BO, vl + V::G1, vl + V::BE1);
            publish();
            __syncthreads();
            if (p.conv_w) {
                // dilated convolutions on the grid (token = cell): three residual units
                // X += ReLU(b_j + sum_{a,e} X[cell + dil_j (a-1, e-1)] Wd_j[a][e]); the k of a
                // unit (nine taps of D) in activation registers, dealt out to the wavefronts
                for (int j = 0; j < 3; ++j) {
                    const float* wj = p.conv_w + ((size_t)l * 3 + j) * (9 * D * D + D);
                    clear(acc);
#pragma unroll 1
                    for (int kg = wave; kg < 36; kg += WAVES) {
                        const int* row = ctab + (j * 9 + kg / 4) * NP;
                        const int k0 = (kg % 4) * KA;
                        f32x4 wc[KA / 4];
                        load_w(wc, wj + kg * KA * D);
                        gemm(acc, wc, [&](int, int r, int k) { return row[r] >= 0 ? X[row[r] + k0 + k] : 0.f; }, nullptr);
                    }
                    store(WP + wave * NP * D, D, acc);
                    __syncthreads();
                    const Own oc;
                    const int f = oc.f, n0 = oc.n0;
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        const int n = n0 + e * TPP;
                        if (n < N) {
                            float y = wj[9 * D * D + f];
#pragma unroll
                            for (int w = 0; w < WAVES; ++w) y += WP[(w * NP + n) * D + f];
                            x[e] += fmaxf(y, 0.f);
                        }
                    }
                    publish();
                    __syncthreads();
                }
            }
            start(acc, vl + V::B1 + cg1 * D, kp1);
            gemm(acc, wa, [&](int, int r, int k) { return X[r * SX + kp1 * S::KQ + k]; }, src_wq(wn));
            store(HP + kp1 * NP * SF + cg1 * D, SF, acc);
            if constexpr (MR == 5) {   // the fifth column group: its k halves to wavefronts 0 .. KP - 1
                if (role < KP) {
                    f32x4 w5[S::KQ / 4];
                    load_w(w5, wl + W1 + 4 * D * D + role * S::KQ * D);
                    start(acc, vl + V::B1 + 4 * D, role);
                    gemm(acc, w5, [&](int, int r, int k) { return X[r * SX + role * S::KQ + k]; }, nullptr);
                    store(HP + role * NP * SF + 4 * D, SF, acc);
                }
            }
            __syncthreads();
            clear(acc);
            gemm(acc, w2, [&](int, int r, int k) {
                const int kk = wave * S::KW2 + k;
                float h = HP[r * SF + kk];
                if constexpr (KP == 2) h += HP[(NP + r) * SF + kk];
                return fmaxf(h, 0.f);
            }, src_w2(wn));
            store(WP + wave * NP * D, D, acc);
            __syncthreads();
            add_norm(vl + V::B2, vl + V::G2, vl + V::BE2);
            if (l + 1 < p.L) {
                publish();
                __syncthreads();
            }
        }
        if (t >= p.in.W - p.readouts) {
            publish();
            __syncthreads();
            readout(t - (p.in.W - p.readouts));
        }
    }
}

template <int D, int MR, int NT>
hipError_t launch_shape(const F32Params& p, hipStream_t s) {
    using S = F32Shape<D, MR, NT>;
    const size_t smem = S::smem(p.L, p.conv_w != nullptr);
    hipError_t e = hipFuncSetAttribute((const void*)f32_window_kernel<D, MR, NT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    f32_window_kernel<D, MR, NT><<<dim3((unsigned)p.in.nwin), dim3(S::THREADS), smem, s>>>(p);
    return hipGetLastError();
}

// The token counts of the distances that fit (8 and 16, 24 and 36, 48 and 64 tokens for d = 3, 5,
// 7) in tiles of TQ tokens: every size the configuration check accepts has its tile count here.
template <int D, int MR>
hipError_t launch_dm(const F32Params& p, hipStream_t s) {
    constexpr int TQ = 256 / D;
    const int nt = (p.ntok + TQ - 1) / TQ;
    if constexpr (D == 64) {
        if (nt == 2) return launch_shape<D, MR, 2>(p, s);
        if (nt == 4) return launch_shape<D, MR, 4>(p, s);
        if (nt == 6) return launch_shape<D, MR, 6>(p, s);
    } else if constexpr (D == 32) {
        if (nt == 1) return launch_shape<D, MR, 1>(p, s);
        if (nt == 2) return launch_shape<D, MR, 2>(p, s);
        if (nt == 3) return launch_shape<D, MR, 3>(p, s);
        if (nt == 5) return launch_shape<D, MR, 5>(p, s);
    } else {
        if (nt == 1) return launch_shape<D, MR, 1>(p, s);
        if (nt == 2) return launch_shape<D, MR, 2>(p, s);
        if (nt == 3) return launch_shape<D, MR, 3>(p, s);
        if (nt == 4) return launch_shape<D, MR, 4>(p, s);
    }
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_d(const F32Params& p, hipStream_t s) {
    if (p.F == 4 * D) return launch_dm<D, 4>(p, s);
    if (p.F == 5 * D) return launch_dm<D, 5>(p, s);
    return hipErrorInvalidValue;
}

}  // namespace

// The size rule of the fp32 configurations (fp32 values of a window: state, Q, K, V, attention
// output, hidden units and scores); the kernel's own tables are smaller than a CU's LDS for all
// of them.
size_t f32_window_smem_bytes(int N, int D, int H, int F) {
    return ((size_t)6 * N * D + (size_t)N * F + (size_t)H * N * N) * sizeof(float);
}

hipError_t launch_f32_window(const F32Params& p, hipStream_t s) {
    if (p.in.nwin <= 0) return hipSuccess;
    switch (p.D) {
        case 16: return launch_d<16>(p, s);
        case 32: return launch_d<32>(p, s);
        case 64: return launch_d<64>(p, s);
        default: return hipErrorInvalidValue;
    }
}
