// The state-resident decoder of resident.hip for few windows: one workgroup per window instead of
// one wavefront, the matrices' output features split over its four wavefronts.
//
// resident_kernel puts a window on one wavefront and four windows on a workgroup: full SIMDs from
// 1024 windows up, but a layer of one window is 400 weight fragments through one wavefront (about
// 25 us at three token blocks) however few windows there are. Here wavefront w owns the 32-feature
// group w of Q, K and V and the attention of its heads, row tiles 2 w, 2 w + 1 of the state (the
// out-projection's and the second feed-forward matrix's outputs) and the hidden k-steps w, w + 4,
// .... A weight fragment is used by exactly one wavefront, so it goes from L2 straight to that
// wavefront's registers, through a ring refilled right behind each use that runs ahead across the
// stages, layers and rounds; what the wavefronts exchange through LDS are the attention output, the
// hidden units and the layer inputs, each as the B fragments of the next product, and the state
// for the LayerNorm statistics.
//
// What bounds it is the chain of stages: eight exchanges with a barrier per layer and one wavefront
// per SIMD, so attention, LayerNorms and the waits at barriers are exposed; the weights themselves,
// 384 KB a layer at the CU's 64 bytes per cycle, are 2.6 us of the 8.3 us a layer takes at 48 tokens
// (a ring of 8, 16, 24 or 32 fragments: 350, 354, 357, 357 us; 8 is also no slower at 8, 24 and 64
// tokens, from 1 to 768 windows). 22 windows of 48 tokens, 14 rounds of 3 layers: 1024 us
// (resident_kernel) to 350 us; 256 windows 1037 to 400 us.
//
// Bit for bit the results of resident_kernel (a window's result does not depend on the batch it
// is in): the same stream, every output element accumulated over k in the same order in one
// accumulator, the attention of a group by the same code, and a block's LayerNorm statistics by
// one wavefront over all features in the same order.
#include "common.h"
#include "kernels.h"
#include "pipeline.h"
#include "residentshape.h"

namespace {

constexpr int SWAVES = RKS;        // wavefronts of a window: one per 32-feature group
constexpr int SRING = 8;           // weight fragments in flight per wavefront

template <int TB, int DH>
__global__ __launch_bounds__(SWAVES * 64, 1) void resident_split_kernel(ResidentParams p) {
    using S = RShape<4>;
    using V = RVec<4>;
    constexpr int FKS = S::F / 32;   // hidden k-steps
    // a wavefront's fragments of one layer: [Q K V | Wo | W1 | W2]
    constexpr int N_WO = S::QKV_FRAGS, N_W1 = N_WO + 2 * RKS, N_W2 = N_W1 + 2 * FKS, N_END = N_W2 + 2 * FKS;
    static_assert(N_END % SRING == 0 && SRING <= N_END, "ring positions repeat every layer");
    static_assert(TB <= SWAVES, "a wavefront for each block's statistics");
    const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t win = blockIdx.x;

    __shared__ __align__(16) uint16_t ys[RKS * TB * FRAG];    // attention output [k-step][block]
    __shared__ __align__(16) uint16_t xbs[RKS * TB * FRAG];   // layer or feed-forward input [k-step][block]
    __shared__ __align__(16) uint16_t hs[FKS * TB * FRAG];    // hidden units [k-step][block]
    __shared__ __align__(16) float xs[TB * RRT * 256];        // state, for the statistics
    __shared__ __align__(16) float vec[RMAXL * V::PER_LAYER];
    __shared__ float stat[TB][2][64];

    bf16x8 a[SRING];
    // fragment n of the layer at fragment `cur` of the stream, or n - N_END of the layer at `nxt`. (The
    // address space is stated because the compiler loses it here: flat loads, and then every wait for
    // LDS waits for the weights in flight too.)
    auto load = [&](int cur, int nxt, auto nc) {
        constexpr int NN = decltype(nc)::value, N = NN % N_END;
        int f;
        if constexpr (N < N_WO) {              // Q, K, V: group `wave`
            f = wave * RCHUNK + N;
        } else if constexpr (N < N_W1) {       // Wo: k-step J / 2, the two owned row tiles
            constexpr int J = N - N_WO;
            f = J / 2 * RCHUNK + S::QKV_FRAGS + 2 * wave + J % 2;
        } else if constexpr (N < N_W2) {       // W1: hidden k-step wave + 4 T, k-step ks, its two row tiles
            constexpr int T = (N - N_W1) / (2 * RKS), J = (N - N_W1) % (2 * RKS);
            f = (RKS + 2 * T + (wave >> 1)) * RCHUNK + J / 2 * (S::CH / 16) + 2 * (wave & 1) + J % 2;
        } else {                               // W2: hidden k-step kk, the two owned row tiles
            constexpr int kk = (N - N_W2) / 2;
            f = (RKS + kk / 2) * RCHUNK + S::W1_FRAGS + kk % 2 * RRT + 2 * wave + N % 2;
        }
        const uint16_t* src = p.stream + (size_t)((NN < N_END ? cur : nxt) + f) * FRAG;
        a[NN % SRING] = __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(1))) u16x8*)(src + lane * 8));
    };
    constexpr int LAYER = S::LAYER_CHUNKS * RCHUNK;
    static_for<SRING>([&](auto nc) { load(0, 0, nc); });

    for (int i = threadIdx.x; i < p.L * V::PER_LAYER; i += SWAVES * 64) vec[i] = p.vecs[i];
    f32x4 s0[2][TB], we[2];   // b_e + PE and w_e of the owned rows
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        we[h] = ld4(p.we + (2 * wave + h) * 16 + 4 * g);
#pragma unroll
        for (int b = 0; b < TB; ++b) s0[h][b] = ld4(p.S0 + ((b * RRT + 2 * wave + h) * 64 + lane) * 4);
    }
    const uint32_t* meas = p.in.meas + win * (p.in.W + 1) * p.in.words;
    const int type = p.in.types[win];
    int stab[TB];   // this lane's token's stabilizer in each block, or -1 (reads word 0)
    uint32_t m_prev[TB], m_cur[TB];   // its measurement words of rows t and t + 1
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int s = b * 16 + col;
        stab[b] = s < p.ntok ? (p.tok_stab ? p.tok_stab[s] : s) : -1;
        const int wd = stab[b] >= 0 ? stab[b] >> 5 : 0;
        m_prev[b] = meas[wd];
        m_cur[b] = meas[p.in.words + wd];
    }
    bf16x4 ones;   // A operand with row 0 all ones: column sums on the matrix core
#pragma unroll
    for (int i = 0; i < 4; ++i) ones[i] = (__bf16)(col == 0 ? 1.0f : 0.0f);

    f32x4 x[2][TB];        // row tiles 2 wave, 2 wave + 1 of the state
    bf16x8 xb[RKS][TB];    // the current product's operand, all features
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < TB; ++b) x[h][b] = f32x4{0.f, 0.f, 0.f, 0.f};   // D_0 = 0

    auto frag = [&](const uint16_t* m, int i) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(m + i * FRAG + lane * 8));
    };
    auto put = [&](uint16_t* m, int i, bf16x8 v) {
        *reinterpret_cast<u16x8*>(m + i * FRAG + lane * 8) = __builtin_bit_cast(u16x8, v);
    };
    // the owned rows, packed, are k-step `wave` of every wavefront's next product
    auto exchange = [&]() {
#pragma unroll
        for (int b = 0; b < TB; ++b) put(xbs, wave * TB + b, pack_b(x[0][b], x[1][b]));
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
            for (int b = 0; b < TB; ++b) xb[ks][b] = frag(xbs, ks * TB + b);
    };
    auto add = [&](const float* v) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 bias = ld4(v + (2 * wave + h) * 16 + 4 * g);
#pragma unroll
            for (int b = 0; b < TB; ++b) x[h][b] += bias;
        }
    };
    // LayerNorm of the owned rows; block b's statistics from wavefront b
    auto normalise = [&](const float* gamma, const float* beta) {
        constexpr float inv_d = 1.0f / RD;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < TB; ++b) *reinterpret_cast<f32x4*>(xs + ((b * RRT + 2 * wave + h) * 64 + lane) * 4) = x[h][b];
        __syncthreads();
        if (wave < TB) {
            f32x4 y[RRT];
            float s = 0.f;
#pragma unroll
            for (int rt = 0; rt < RRT; ++rt) y[rt] = ld4(xs + ((wave * RRT + rt) * 64 + lane) * 4);
#pragma unroll
            for (int rt = 0; rt < RRT; ++rt) s += (y[rt][0] + y[rt][1]) + (y[rt][2] + y[rt][3]);
            const float mean = group_sum(s) * inv_d;
            float v = 0.f;
#pragma unroll
            for (int rt = 0; rt < RRT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float c = y[rt][i] - mean;
                    v = fmaf(c, c, v);
                }
            stat[wave][0][lane] = mean;
            stat[wave][1][lane] = rsqrtf(group_sum(v) * inv_d + p.eps);
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 gm = ld4(gamma + (2 * wave + h) * 16 + 4 * g), bt = ld4(beta + (2 * wave + h) * 16 + 4 * g);
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const float mean = stat[b][0][lane], rstd = stat[b][1][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[h][b][i] = fmaf((x[h][b][i] - mean) * rstd, gm[i], bt[i]);
            }
        }
    };

    for (int t = 0; t < p.in.W; ++t) {
        // ---- embedding of round t folded into the state: X = kappa (E_t w_e + b_e + PE + X)
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const uint32_t w = event_from(m_prev[b], m_cur[b], t, type, p.in.b_left, p.in.d);
            const float ev = stab[b] >= 0 ? (float)((w >> (stab[b] & 31)) & 1u) : 0.f;
            const bool real = b * 16 + col < p.ntok;
            m_prev[b] = m_cur[b];
            if (t + 2 <= p.in.W) m_cur[b] = meas[(t + 2) * p.in.words + (stab[b] >= 0 ? stab[b] >> 5 : 0)];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[h][b][i] = p.kappa * ((real ? ev * we[h][i] + s0[h][b][i] : 0.f) + x[h][b][i]);
        }
        for (int l = 0; l < p.L; ++l) {
            const float* vl = vec + l * V::PER_LAYER;
            const int cur = l * LAYER, nxt = l + 1 < p.L ? cur + LAYER : 0;
            // fragments FROM .. FROM + COUNT - 1: use(j, fragment), each replaced behind its use
            auto run = [&](auto fromc, auto countc, const auto& use) {
                constexpr int FROM = decltype(fromc)::value;
                static_for<decltype(countc)::value>([&](auto jc) {
                    constexpr int N = FROM + decltype(jc)::value;
                    use(jc, a[N % SRING]);
                    __builtin_amdgcn_sched_barrier(0);
                    load(cur, nxt, std::integral_constant<int, N + SRING>{});
                });
            };
            exchange();

            // ---- Q, K, V of group `wave` and the attention of its heads
            {
                f32x4 q[2][TB], k[2][TB], v[2][TB];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int f0 = wave * 32 + hh * 16;
                    const f32x4 bq = ld4(vl + V::BQ + f0 + 4 * g), bk = ld4(vl + V::BK + f0 + 4 * g);
                    const float bvv = vl[V::BV + f0 + col];   // V tiles: features along columns
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        q[hh][b] = bq;
                        k[hh][b] = bk;
                        v[hh][b] = f32x4{bvv, bvv, bvv, bvv};
                    }
                }
                run(std::integral_constant<int, 0>{}, std::integral_constant<int, S::QKV_FRAGS>{}, [&](auto jc, const bf16x8& w) {
                    constexpr int J = decltype(jc)::value, part = J / (2 * RKS), ks = J / 2 % RKS, hh = J % 2;
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        if constexpr (part == 0) q[hh][b] = mfma16x16x32(w, xb[ks][b], q[hh][b]);
                        else if constexpr (part == 1) k[hh][b] = mfma16x16x32(w, xb[ks][b], k[hh][b]);
                        else v[hh][b] = mfma16x16x32(xb[ks][b], w, v[hh][b]);
                    }
                });
                bf16x8 y[TB];
                attend_group<TB, DH>(q, k, v, y, p.qscale, p.ntok, g, ones);
#pragma unroll
                for (int b = 0; b < TB; ++b) put(ys, wave * TB + b, y[b]);
            }
            __syncthreads();

            // ---- out-projection into the owned rows (the residual is the state itself), LayerNorm 1
            bf16x8 yb[RKS][TB];
#pragma unroll
            for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
                for (int b = 0; b < TB; ++b) yb[ks][b] = frag(ys, ks * TB + b);
            run(std::integral_constant<int, N_WO>{}, std::integral_constant<int, 2 * RKS>{}, [&](auto jc, const bf16x8& w) {
                constexpr int J = decltype(jc)::value;
#pragma unroll
                for (int b = 0; b < TB; ++b) x[J % 2][b] = mfma16x16x32(w, yb[J / 2][b], x[J % 2][b]);
            });
            add(vl + V::BO);
            normalise(vl + V::G1, vl + V::BE1);
            exchange();
            add(vl + V::B2);   // the accumulators of the second matrix start here

            // ---- feed-forward
            static_for<FKS / RKS>([&](auto tc) {
                constexpr int T = decltype(tc)::value;
                const int kk = wave + RKS * T;
                f32x4 h[2][TB];
#pragma unroll
                for (int rh = 0; rh < 2; ++rh) {
                    const f32x4 b1 = ld4(vl + V::B1 + kk * 32 + rh * 16 + 4 * g);
#pragma unroll
                    for (int b = 0; b < TB; ++b) h[rh][b] = b1;
                }
                run(std::integral_constant<int, N_W1 + T * 2 * RKS>{}, std::integral_constant<int, 2 * RKS>{},
                    [&](auto jc, const bf16x8& w) {
                        constexpr int J = decltype(jc)::value;
#pragma unroll
                        for (int b = 0; b < TB; ++b) h[J % 2][b] = mfma16x16x32(w, xb[J / 2][b], h[J % 2][b]);
                    });
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    f32x4 lo = h[0][b], hi = h[1][b];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        lo[i] = fmaxf(lo[i], 0.f);
                        hi[i] = fmaxf(hi[i], 0.f);
                    }
                    put(hs, kk * TB + b, pack_b(lo, hi));
                }
            });
            __syncthreads();
            // hidden fragments two k-steps ahead of their products
            bf16x8 hb[3][TB];
            auto read_h = [&](auto kc) {
                constexpr int K = decltype(kc)::value;
                if constexpr (K < FKS)
#pragma unroll
                    for (int b = 0; b < TB; ++b) hb[K % 3][b] = frag(hs, K * TB + b);
            };
            read_h(std::integral_constant<int, 0>{});
            read_h(std::integral_constant<int, 1>{});
            run(std::integral_constant<int, N_W2>{}, std::integral_constant<int, 2 * FKS>{}, [&](auto jc, const bf16x8& w) {
                constexpr int J = decltype(jc)::value, K = J / 2;
                if constexpr (J % 2 == 0) read_h(std::integral_constant<int, K + 2>{});
#pragma unroll
                for (int b = 0; b < TB; ++b) x[J % 2][b] = mfma16x16x32(w, hb[K % 3][b], x[J % 2][b]);
            });
            normalise(vl + V::G2, vl + V::BE2);
        }
    }

    // the final state D_W for the readout
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < TB; ++b)
            *reinterpret_cast<f32x4*>(p.X + (((win * p.nbw + b) * RRT + 2 * wave + h) * 64 + lane) * 4) = x[h][b];
}

template <int TB>
hipError_t launch_tb(int dh, const ResidentParams& p, hipStream_t s) {
    const dim3 grid((unsigned)p.in.nwin), block(SWAVES * 64);
    if (dh == 16) resident_split_kernel<TB, 16><<<grid, block, 0, s>>>(p);
    else if (dh == 32) resident_split_kernel<TB, 32><<<grid, block, 0, s>>>(p);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_resident_split(int mr, int dh, const ResidentParams& p, hipStream_t s) {
    if (p.in.nwin <= 0) return hipSuccess;
    if (mr != 4 || p.L > RMAXL) return hipErrorInvalidValue;
    switch (p.nbw) {
        case 1: return launch_tb<1>(dh, p, s);
        case 2: return launch_tb<2>(dh, p, s);
        case 3: return launch_tb<3>(dh, p, s);
        case 4: return launch_tb<4>(dh, p, s);
        default: return hipErrorInvalidValue;
    }
}
