// The token-local stages of tok.hip for small batches: the same arithmetic, split the other way.
//
// tok_kernel gives a wavefront 32 whole tokens and lets four wavefronts share one weight stream
// through LDS: the right split when there are enough tokens for every CU, but a workgroup then
// takes 128 tokens and walks the whole stream (48 chunks with a barrier each at d_model 256), and
// a few windows occupy a few CUs. Here a workgroup takes one or two 16-token blocks, and its
// D / 32 wavefronts split every matrix's output features: wavefront w owns 32 features of the
// state (row tiles 2 w, 2 w + 1, which are k-step w of the next product), the feed-forward's
// hidden k-steps w, w + KS, ..., and 32 features each of Q, K and V. A weight fragment is used by
// exactly one wavefront, so it goes from L2 straight to that wavefront's registers, through a ring
// of 2 KS fragments refilled right behind its use and running ahead across the stages; what the
// wavefronts exchange through LDS are the activations, as the B fragments of the next product.
// What bounds it is the CU's 64 bytes per cycle from L1 (150 GB/s measured for one workgroup
// alone): 1.5 MB of weights at d_model 256, about 10 us, against 5 us of matrix work for two blocks;
// more tokens per workgroup would not fit LDS. Post + QKV launch at d_model 256: 22 us for 78 blocks,
// 24 us for 312 (tok_kernel 46 and 48); by time stamps in one workgroup 5.4 K cycles pass before
// its first operands are in, the two feed-forward matrices run at 57 bytes per cycle, a LayerNorm
// with its exchanges takes 2.5 K, and the rest is launch. Warming L2 with the weights beforehand,
// from this kernel's start or from the attention before it, changed nothing.
//
// Bit for bit the results of tok_kernel (a window's result does not depend on the batch it is
// in): every output element accumulates over k in the same order in one accumulator, and the
// LayerNorm statistics of a block are computed by one wavefront over all features in the order
// tok_kernel uses.
#include "common.h"
#include "kernels.h"
#include "pipeline.h"
#include "tokshape.h"

hipError_t launch_wide_4(int D, int flags, const TokParams& p, int64_t n_tb, hipStream_t s);
hipError_t launch_wide_5(int D, int flags, const TokParams& p, int64_t n_tb, hipStream_t s);

namespace {

template <int D, int MR, int FLAGS, int TB>
__global__ __launch_bounds__(D * 2, 2) void wide_kernel(TokParams p) {
    using S = Shape<D, 4, MR>;
    using V = Vecs<D, S::F>;
    constexpr int RT = S::RT, KS = S::KS, CH = S::CH, F = S::F, FKS = F / 32, THREADS = KS * 64;
    constexpr bool WO_ONLY = (FLAGS & TOK_WO) != 0, FFN_ONLY = (FLAGS & TOK_FFN) != 0;
    constexpr bool DO_WO = (FLAGS & TOK_POST) != 0 || WO_ONLY, DO_FFN = (FLAGS & TOK_POST) != 0 || FFN_ONLY;
    constexpr bool POST = DO_WO || DO_FFN, QKV = (FLAGS & TOK_QKV) != 0, RES = (FLAGS & TOK_RESNET) != 0;
    const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tb0 = (int64_t)blockIdx.x * TB;

    __shared__ __align__(16) float xs[TB * RT * 256];            // state, for the statistics
    __shared__ __align__(16) uint16_t xbs[KS * TB * FRAG];       // the product's operand [k-step][block]
    __shared__ __align__(16) uint16_t hs[DO_FFN ? FKS * TB * FRAG : 8];   // hidden units [k-step][block]
    __shared__ __align__(16) float vec[V::SIZE];
    __shared__ float stat[TB][2][64];

    // ---- the weight ring: iteration i of the sequence [Wo | W1 x MR | W2 x MR | Q K V] uses 2 KS
    // fragments of this wavefront; fragment j of the next iteration replaces fragment j after use
    constexpr int RING = 2 * KS;
    constexpr int I_W1 = DO_WO ? 1 : 0, I_W2 = I_W1 + (DO_FFN ? MR : 0), I_QKV = I_W2 + (DO_FFN ? MR : 0);
    constexpr int I_END = I_QKV + (QKV ? 3 : 0);
    constexpr int WOF = RT * KS, KC = CH / 32, NW1 = (CH / 16) * KS;   // Wo fragments; k-steps and W1 fragments of a chunk
    bf16x8 a[RING];
    auto load = [&](auto ic, auto jc) {
        constexpr int I = decltype(ic)::value, J = decltype(jc)::value;
        if constexpr (I < I_END) {
            const uint16_t* src;
            if constexpr (I < I_W1) {                     // Wo: row tiles 2 wave, 2 wave + 1
                src = p.post_stream + (size_t)(2 * wave * KS + J) * FRAG;
            } else if constexpr (I < I_W2) {              // W1: the two row tiles of hidden k-step kk
                const int kk = wave + KS * (I - I_W1);
                src = p.post_stream + (size_t)(WOF + kk / KC * 32 + kk % KC * 2 * KS + J) * FRAG;
            } else if constexpr (I < I_QKV) {             // W2: k-steps KS (I - I_W2) .., both row tiles
                constexpr int kk = KS * (I - I_W2) + J / 2;
                src = p.post_stream + (size_t)(WOF + kk / KC * 32 + NW1 + (2 * wave + J % 2) * KC + kk % KC) * FRAG;
            } else {                                      // Q, K, V: output group wave of each
                src = p.qkv_stream + (size_t)((wave + KS * (I - I_QKV)) * 2 * KS + J) * FRAG;
            }
            a[J] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(src + lane * 8));
        }
    };
    // iteration I: use(j, fragment) for each, reloading behind it
    auto iteration = [&](auto ic, const auto& use) {
        constexpr int I = decltype(ic)::value;
        static_for<RING>([&](auto jc) {
            use(jc, a[decltype(jc)::value]);
            __builtin_amdgcn_sched_barrier(0);
            load(std::integral_constant<int, I + 1>{}, jc);
        });
    };

    // ---- loads: the attention output (one k-step per wavefront), the owned rows of the state, the
    // first fragments, the vectors
    f32x4 x[2][TB];   // row tiles 2 wave + h
    u16x8 y[TB];
    if constexpr (DO_WO) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
            y[b] = *reinterpret_cast<const u16x8*>(p.Y + (((tb0 + b) * KS + wave) * 64 + lane) * 8);
    }
    if constexpr (POST) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < TB; ++b) x[h][b] = ld4(p.X + (((tb0 + b) * RT + 2 * wave + h) * 64 + lane) * 4);
    }
    static_for<RING>([&](auto jc) { load(std::integral_constant<int, 0>{}, jc); });
    {
        constexpr int NP_V = POST ? V::BQKV / 4 : 0, NQ_V = QKV ? V::QKV_VECS / 4 : 0;
        for (int k = threadIdx.x; k < NP_V + NQ_V; k += THREADS) {
            const float* src = k < NP_V ? p.post_vecs + k * 4 : p.bqkv + (k - NP_V) * 4;
            *reinterpret_cast<f32x4*>(vec + (k < NP_V ? k * 4 : V::BQKV + (k - NP_V) * 4)) = ld4(src);
        }
    }
    float ev[TB];
    int row[TB];
    if constexpr ((FLAGS & TOK_EMBED) != 0) {
#pragma unroll
        for (int b = 0; b < TB; ++b) token_event<RES>(p, tb0 + b, col, ev[b], row[b]);
    }

    bf16x8 xb[KS][TB];   // every wavefront's operand, read back from LDS
    auto gather = [&]() {
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int b = 0; b < TB; ++b)
                xb[ks][b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(xbs + (ks * TB + b) * FRAG + lane * 8));
    };
    auto publish = [&](int b, u16x8 v) { *reinterpret_cast<u16x8*>(xbs + (wave * TB + b) * FRAG + lane * 8) = v; };
    // the owned rows, packed, are k-step `wave` of the next product
    auto exchange = [&]() {
#pragma unroll
        for (int b = 0; b < TB; ++b) publish(b, __builtin_bit_cast(u16x8, pack_b(x[0][b], x[1][b])));
        gather();
    };
    // LayerNorm of the owned rows; block b's statistics from wavefront b
    auto normalise = [&](const float* gamma, const float* beta) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < TB; ++b) *reinterpret_cast<f32x4*>(xs + ((b * RT + 2 * wave + h) * 64 + lane) * 4) = x[h][b];
        __syncthreads();
        if (wave < TB) {
            f32x4 v[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) v[rt] = ld4(xs + ((wave * RT + rt) * 64 + lane) * 4);
            float mean, rstd;
            ln_stats<RT>([&](int rt) -> const f32x4& { return v[rt]; }, p.eps, mean, rstd);
            stat[wave][0][lane] = mean;
            stat[wave][1][lane] = rstd;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 gm = ld4(gamma + (2 * wave + h) * 16 + 4 * g), bt = ld4(beta + (2 * wave + h) * 16 + 4 * g);
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const float mean = stat[b][0][lane], rstd = stat[b][1][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[h][b][i] = ln_apply(x[h][b][i], mean, rstd, gm[i], bt[i]);
            }
        }
    };
    auto add_bias = [&](const float* v) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 bias = ld4(v + (2 * wave + h) * 16 + 4 * g);
#pragma unroll
            for (int b = 0; b < TB; ++b) x[h][b] += bias;
        }
    };

    if constexpr (DO_WO) {
#pragma unroll
        for (int b = 0; b < TB; ++b) publish(b, y[b]);
        gather();
        iteration(std::integral_constant<int, 0>{}, [&](auto jc, const bf16x8& w) {
            constexpr int J = decltype(jc)::value;
#pragma unroll
            for (int b = 0; b < TB; ++b) x[J / KS][b] = mfma16x16x32(w, xb[J % KS][b], x[J / KS][b]);
        });
        add_bias(vec + V::BO);
        normalise(vec + V::G1, vec + V::BE1);
    }
    if constexpr (WO_ONLY) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
            *reinterpret_cast<u16x8*>(p.G + ((((tb0 + b) * 16 + col) * KS + wave) * 4 + g) * 8) =
                __builtin_bit_cast(u16x8, pack_b(x[0][b], x[1][b]));
    }
    if constexpr (DO_FFN) {
        exchange();
        add_bias(vec + V::B2);   // the accumulators of the second matrix start here
        static_for<MR>([&](auto tc) {
            constexpr int T = decltype(tc)::value;
            const int kk = wave + KS * T;
            f32x4 h[2][TB];
#pragma unroll
            for (int rh = 0; rh < 2; ++rh) {
                const f32x4 bias = ld4(vec + V::B1 + kk * 32 + rh * 16 + 4 * g);
#pragma unroll
                for (int b = 0; b < TB; ++b) h[rh][b] = bias;
            }
            iteration(std::integral_constant<int, I_W1 + T>{}, [&](auto jc, const bf16x8& w) {
                constexpr int J = decltype(jc)::value;
#pragma unroll
                for (int b = 0; b < TB; ++b) h[J / KS][b] = mfma16x16x32(w, xb[J % KS][b], h[J / KS][b]);
            });
#pragma unroll
            for (int b = 0; b < TB; ++b)
                *reinterpret_cast<u16x8*>(hs + (kk * TB + b) * FRAG + lane * 8) =
                    __builtin_bit_cast(u16x8, pack_b(relu4(h[0][b]), relu4(h[1][b])));
        });
        __syncthreads();
        // hidden fragments two k-steps ahead of their products
        bf16x8 hb[3][TB];
        auto read_h = [&](auto kc) {
            constexpr int K = decltype(kc)::value;
            if constexpr (K < FKS)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    hb[K % 3][b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(hs + (K * TB + b) * FRAG + lane * 8));
        };
        read_h(std::integral_constant<int, 0>{});
        read_h(std::integral_constant<int, 1>{});
        static_for<MR>([&](auto tc) {
            constexpr int T = decltype(tc)::value;
            iteration(std::integral_constant<int, I_W2 + T>{}, [&](auto jc, const bf16x8& w) {
                constexpr int J = decltype(jc)::value, K = KS * T + J / 2;
                if constexpr (J % 2 == 0) read_h(std::integral_constant<int, K + 2>{});
#pragma unroll
                for (int b = 0; b < TB; ++b) x[J % 2][b] = mfma16x16x32(w, hb[K % 3][b], x[J % 2][b]);
            });
        });
        normalise(vec + V::G2, vec + V::BE2);
    }
    if constexpr (DO_FFN && (FLAGS & TOK_EMBED) != 0) {
        if (p.state_out) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    *reinterpret_cast<u16x4*>(p.state_out + (((tb0 + b) * RT + 2 * wave + h) * 64 + lane) * 4) = to_bf16x4(x[h][b]);
        }
    }
    if constexpr ((FLAGS & TOK_EMBED) != 0) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int blk = (int)((tb0 + b) % p.nbw);
            const bool real = blk * 16 + col < p.ntok;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int rt = 2 * wave + h;
                f32x4 s0 = ld4(p.S0 + (((int64_t)blk * RT + rt) * 64 + lane) * 4);
                const f32x4 we = ld4(p.we + rt * 16 + 4 * g);
                if constexpr (RES) s0 += ld4(p.emb_tab + (size_t)row[b] * D + rt * 16 + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) x[h][b][i] = fold(real, ev[b], we[i], s0[i], POST ? x[h][b][i] : 0.f, p.kappa);
            }
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < TB; ++b)
            *reinterpret_cast<f32x4*>(p.X + (((tb0 + b) * RT + 2 * wave + h) * 64 + lane) * 4) = x[h][b];

    if constexpr (QKV) {
        exchange();   // (its barrier publishes the biases too where no other came before)
        static_for<3>([&](auto pc) {
            constexpr int PART = decltype(pc)::value;
            const int og = wave + KS * PART;
            f32x4 q[2][TB];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                f32x4 bias;
                if constexpr (PART == 2) {   // V: one column value per lane
                    const float bv = vec[V::BV + (wave * 32 + hh * 16 + col) * V::REP];
                    bias = f32x4{bv, bv, bv, bv};
                } else {
                    bias = ld4(vec + V::BQKV + og * 32 + hh * 16 + 4 * g);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b) q[hh][b] = bias;
            }
            iteration(std::integral_constant<int, I_QKV + PART>{}, [&](auto jc, const bf16x8& w) {
                constexpr int J = decltype(jc)::value;   // k-step J / 2, row tile J % 2
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    if constexpr (PART == 2) q[J % 2][b] = mfma16x16x32(xb[J / 2][b], w, q[J % 2][b]);
                    else q[J % 2][b] = mfma16x16x32(w, xb[J / 2][b], q[J % 2][b]);
                }
            });
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                uint16_t* dst = p.QKV + ((tb0 + b) * (3 * KS) + og) * FRAG;
                if constexpr (PART == 2) {
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2)
                        *reinterpret_cast<u16x4*>(dst + h2 * (FRAG / 2) + lane * 4) = to_bf16x4(q[h2][b]);
                } else {
                    const float sc = PART == 0 ? p.qscale : 1.0f;   // Q: log2(e)/sqrt(dh)
                    *reinterpret_cast<u16x8*>(dst + lane * 8) = __builtin_bit_cast(u16x8, pack_b(q[0][b] * sc, q[1][b] * sc));
                }
            }
        });
    }
}

template <int D, int MR, int TB>
hipError_t launch_wide_d(int flags, const TokParams& p, int64_t n_tb, hipStream_t s) {
    const dim3 grid((unsigned)((n_tb + TB - 1) / TB)), block(D * 2);
    switch (flags) {
        case TOK_EMBED | TOK_QKV: wide_kernel<D, MR, TOK_EMBED | TOK_QKV, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_POST | TOK_QKV: wide_kernel<D, MR, TOK_POST | TOK_QKV, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_POST | TOK_EMBED | TOK_QKV: wide_kernel<D, MR, TOK_POST | TOK_EMBED | TOK_QKV, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_POST: wide_kernel<D, MR, TOK_POST, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_EMBED | TOK_QKV | TOK_RESNET: wide_kernel<D, MR, TOK_EMBED | TOK_QKV | TOK_RESNET, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_POST | TOK_EMBED | TOK_QKV | TOK_RESNET:
            wide_kernel<D, MR, TOK_POST | TOK_EMBED | TOK_QKV | TOK_RESNET, TB><<<grid, block, 0, s>>>(p);
            break;
        case TOK_WO: wide_kernel<D, MR, TOK_WO, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_FFN | TOK_QKV: wide_kernel<D, MR, TOK_FFN | TOK_QKV, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_FFN | TOK_EMBED | TOK_QKV: wide_kernel<D, MR, TOK_FFN | TOK_EMBED | TOK_QKV, TB><<<grid, block, 0, s>>>(p); break;
        case TOK_FFN | TOK_EMBED | TOK_QKV | TOK_RESNET:
            wide_kernel<D, MR, TOK_FFN | TOK_EMBED | TOK_QKV | TOK_RESNET, TB><<<grid, block, 0, s>>>(p);
            break;
        case TOK_FFN: wide_kernel<D, MR, TOK_FFN, TB><<<grid, block, 0, s>>>(p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D, int MR>
hipError_t launch_wide_tb(int flags, const TokParams& p, int64_t n_tb, hipStream_t s) {
    // one block per workgroup while that still leaves a CU for each
    return n_tb <= 256 ? launch_wide_d<D, MR, 1>(flags, p, n_tb, s) : launch_wide_d<D, MR, 2>(flags, p, n_tb, s);
}

}  // namespace

// Compiled in two parts (WIDE_PART 0 and 1, by feed-forward ratio; both at once without it).
#if !defined(WIDE_PART) || WIDE_PART == 0
hipError_t launch_wide_4(int D, int flags, const TokParams& p, int64_t n_tb, hipStream_t s) {
    return D == 256 ? launch_wide_tb<256, 4>(flags, p, n_tb, s) : launch_wide_tb<128, 4>(flags, p, n_tb, s);
}
#endif
#if !defined(WIDE_PART) || WIDE_PART == 1
hipError_t launch_wide_5(int D, int flags, const TokParams& p, int64_t n_tb, hipStream_t s) {
    return D == 256 ? launch_wide_tb<256, 5>(flags, p, n_tb, s) : launch_wide_tb<128, 5>(flags, p, n_tb, s);
}

hipError_t launch_wide(int D, int F, int flags, const TokParams& p, int64_t n_tb, hipStream_t s) {
    if (n_tb <= 0) return hipSuccess;
    if (D != 128 && D != 256) return hipErrorInvalidValue;
    if (F == 4 * D) return launch_wide_4(D, flags, p, n_tb, s);
    if (F == 5 * D) return launch_wide_5(D, flags, p, n_tb, s);
    return hipErrorInvalidValue;
}
#endif
