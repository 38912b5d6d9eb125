// Projections with few row tiles per workgroup (at most two): Wo, down, the QKV projection of models up to the 8B shape, the
// exit-head transform, and every projection and the vocabulary pass of small models.     out[t][n] = sum_k W[n][k] * act[t][k],  m <= 8 tokens
//
// Such a launch lasts 3 to 25 us, and what it spends beyond reading its weights is a chain: argument fetch, first
// loads, products, sum over the wavefronts, store.  A wavefront issues an instruction every 5 cycles or so (16 wavefronts
// on a compute unit: every 16), so 400 instructions on that chain are a microsecond, and this kernel is written for few of them:
// 8 wavefronts, each with a contiguous run of k-steps of all the workgroup's rows, straight-line loads with constant offsets, no
// masks on tokens past the call's (a column of the product depends on its own column of the operand only, and is not stored),
// the sum over the wavefronts by one wavefront per 8 rows.
//
// Rows are dealt in halves of a tile (8 rows: 128 bytes of each of the tile's four lane groups, whole cache lines), H = 2, 3 or 4
// halves per workgroup (in whole tiles the 13B shape's 320 tiles are two each on 160 of 256 compute units).  Three halves are one
// tile and the lower or upper half of a neighbour; one load fetches the half tile's rows of two k-steps, the lanes of operand
// rows 8..15 taking the second, and two products use one half of the result each.
//
// Layer step, against the kernels this replaces (2500 to 8700 instructions, 16 or 8 wavefronts; here 850 to 1900): 8B shape, bf16,
// context 4096, 1 row 97.2 -> 92.4 us (QKV 13.0 -> 10.4, Wo 9.9 -> 7.9, down 21.7 -> 19.7), context 9203, 8 rows 122.1 -> 113.5; 13B shape, 2
// rows 136.6 -> 129.8 (Wo 14.0 -> 12.3, down 32.0 -> 24.5); tiny fp32 model, a token 136 -> 100 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_launch.h"
#include "ad_proj_device.h"

namespace ad {

namespace {

// k-steps per batch of loads; two batches are in flight.  A wavefront of at most four k-steps (K <= 1024) takes batches of two: a
// batch that it cannot fill repeats its last k-step, and with batches of 8 the 16-bit kernels of the tiny models took 6 us each.
constexpr int proj_batch(int npl) { return npl == 1 ? 8 : 2; }
constexpr int kProjSmallBatch = 2;
constexpr int proj_slots(int h) { return (h + 1) / 2; }         // blocks of 8 tokens x 16 rows a wavefront leaves behind
constexpr size_t proj_lds_bytes(int h, bool from_x) {
    return (size_t)kProjWaves * (from_x ? kStripBytes : proj_slots(h) * 512) + kProjWaves * 8 * 4;
}

// NPL: planes of a weight tile (fp32 models three).  H: halves of a row tile per workgroup.  U: k-steps per batch.  FROM_X: the activations are fp32 rows
// (times a norm weight, with 1 / rms applied to the result), else a packed block, with or without sums of squares for 1 / rms.
template <int NPL, int H, int U, bool F16, bool FROM_X>
__global__ void __launch_bounds__(kProjThreads, 2) k_proj(const void *W, const void *act, const void *norm_w, uint64_t nt_kt, uint64_t k_m, uint64_t ldx_n, GemmOut rest) {
    ProjArgs g;
    (GemmOut &)g = rest;
    g.W = W; g.x = (const float *)act; g.B = act; g.norm_w = norm_w;
    g.NT = (int)nt_kt; g.KT = (int)(nt_kt >> 32); g.K = (int)k_m; g.m = (int)(k_m >> 32); g.ldx = (int)ldx_n; g.N = (int)(ldx_n >> 32);
    const KernelArgLines<48 + sizeof(GemmOut)> lines;
    constexpr int NF = H / 2, NS = proj_slots(H), TB = NPL * 1024;   // whole tiles, slots, bytes of a tile
    constexpr bool HALF = H & 1;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, gq = lane >> 4;
    constexpr int WB = FROM_X ? kStripBytes : NS * 512;         // bytes of a wavefront's part of the LDS
    float *ssq_part = (float *)(lds_raw + kProjWaves * WB);

    const int u0 = blockIdx.x * H, KT = g.KT, last_tile = g.NT - 1;
    const int full0 = (u0 + 1) >> 1;                            // the whole tiles; the half one lies before or after them
    const int upper = u0 & 1;                                   // (H = 3) the half tile is its tile's upper half
    const int half_tile = upper ? full0 - 1 : full0 + NF;
    // the wavefront's k-steps [ka, kb): pairs of them where a load covers two
    int ka, kb;
    if (HALF) {
        const int kp = (KT + 1) >> 1;
        ka = 2 * ((kp * wave) / kProjWaves);
        kb = 2 * ((kp * (wave + 1)) / kProjWaves);
        kb = kb < KT ? kb : KT;
    } else {
        ka = (KT * wave) / kProjWaves;
        kb = (KT * (wave + 1)) / kProjWaves;
    }
    // k-steps that a batch may load: its own, past them the last one again (or, without any, some valid one)
    const int k_ok = kb > ka ? kb - 1 : (ka < KT ? ka : KT - 1);

    // weights: uniform base, 32-bit byte offsets (a packed matrix has less than 4 GiB)
    const char *Wb = (const char *)g.W;
    unsigned wf[NF], wh = 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int t = full0 + f < last_tile ? full0 + f : last_tile;
        wf[f] = (unsigned)t * (unsigned)KT * (unsigned)TB + (unsigned)lane * 16u;
    }
    const int hi_row = (lane >> 3) & 1;                         // this lane's operand row is in 8..15
    if (HALF) {
        const int t = half_tile < last_tile ? half_tile : last_tile;
        wh = (unsigned)t * (unsigned)KT * (unsigned)TB + (unsigned)((lane & 48) + upper * 8 + (lane & 7)) * 16u;
    }
    struct Tiles { bf16x8 f[NF][U][NPL], h[HALF ? U / 2 : 1][NPL]; };
    auto load_w = [&](Tiles &a, int k) {
        if (k + U <= kb) {
            const unsigned o = (unsigned)k * TB;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const char *p = Wb + (size_t)(wf[f] + o);
#pragma unroll
                for (int j = 0; j < U; ++j)
#pragma unroll
                    for (int q = 0; q < NPL; ++q) a.f[f][j][q] = load_weights(p + j * TB + q * 1024);
            }
            if (HALF) {
                const char *p = Wb + (size_t)(wh + o + (unsigned)hi_row * TB);
#pragma unroll
                for (int j = 0; j < U / 2; ++j)
#pragma unroll
                    for (int q = 0; q < NPL; ++q) a.h[j][q] = load_weights(p + 2 * j * TB + q * 1024);
            }
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const unsigned o = (unsigned)(k + j < k_ok ? k + j : k_ok) * TB;
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int q = 0; q < NPL; ++q) a.f[f][j][q] = load_weights(Wb + (size_t)(wf[f] + o) + q * 1024);
            }
            if (HALF) {
#pragma unroll
                for (int j = 0; j < U / 2; ++j) {
                    const int kk = k + 2 * j + hi_row;
                    const unsigned o = wh + (unsigned)(kk < k_ok ? kk : k_ok) * TB;
#pragma unroll
                    for (int q = 0; q < NPL; ++q) a.h[j][q] = load_weights(Wb + (size_t)o + q * 1024);
                }
            }
        }
    };
    // activations: lanes of tokens past the call's read token 0's (the same cache lines)
    const unsigned bo = (unsigned)((n & 7) < g.m ? (n & 7) : 0) * (unsigned)KT * 128u + (unsigned)((n >> 3) * 64 + gq * 16);
    auto load_b = [&](bf16x8 (&b)[U], int k) {
        const char *B = (const char *)g.B;
        if (k + U <= kb) {
            const char *p = B + (size_t)(bo + (unsigned)k * 128u);
#pragma unroll
            for (int j = 0; j < U; ++j) b[j] = *(const bf16x8 *)(p + j * 128);
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) b[j] = *(const bf16x8 *)(B + (bo + (unsigned)(k + j < k_ok ? k + j : k_ok) * 128u));
        }
    };
    // k-steps go to two accumulators in turn: sums half as long (fp16 models show the difference: four layers of the 8B shape, rows
    // 2.09e-7 off with one, 1.88e-7 with two)
    f32x4 acc[NF][2], acch[2];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f][0] = acc[f][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    acch[0] = acch[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto mma_step = [&](const Tiles &a, const bf16x8 (&b)[U], int j) {
#pragma unroll
        for (int q = 0; q < NPL; ++q) {
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f][j & 1] = mma16<F16>(a.f[f][j][q], b[j], acc[f][j & 1]);
            if (HALF) acch[j & 1] = mma16<F16>(a.h[j / 2][q], b[j], acch[j & 1]);
        }
    };
    auto mma = [&](const Tiles &a, const bf16x8 (&b)[U], int k) {
        if (k + U <= kb) {
#pragma unroll
            for (int j = 0; j < U; ++j) mma_step(a, b, j);
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (k + j < kb) mma_step(a, b, j);
        }
    };

    // an output of the epilogue: wavefront h takes half h of the workgroup's rows (SwiGLU: tile h), lane = token * 8 + row
    const int et = lane >> 3, ei = lane & 7, unit = u0 + wave, row = unit * 8 + ei;
    const bool on = wave < H && et < g.m && row < g.N;
    float resid = 0.f, next_w = 0.f;
    auto load_resid = [&]() {
        if (g.epi == EPI_RESID && on) {
            resid = g.resid[(size_t)et * g.ld + row];
            if (g.Bnext) next_w = NPL == 3 ? ((const float *)g.next_norm_w)[row] : from16<F16>(((const uint16_t *)g.next_norm_w)[row]);
        }
    };

    Tiles a0, a1;
    bf16x8 b0[U], b1[U];
    if constexpr (FROM_X) {
        operand_from_rows<NPL, 2 * U, F16>(
            g, ka, kb, lane, (uint16_t *)(lds_raw + wave * WB), ssq_part + wave * 8,
            [&]() {
                load_w(a0, ka);
                if (ka + U < kb) load_w(a1, ka + U);
                lines.use();
            },
            [&](int j, bf16x8 v) {
                if (j < U) b0[j % U] = v;
                else b1[j % U] = v;
            });
        mma(a0, b0, ka);
        mma(a1, b1, ka + U);
    } else {
        load_b(b0, ka);
        load_w(a0, ka);
        if (ka + U < kb) {
            load_b(b1, ka + U);
            load_w(a1, ka + U);
        }
        lines.use();
        load_resid();
        if (g.ssq_in) sum_ssq(g, wave, lane, ssq_part);
        // While four whole batches remain, the loads of the loop are unconditional, so that each product waits for its own
        // operands only.
        int k = ka;
#pragma nounroll
        for (; k + 4 * U <= kb; k += 2 * U) {
            mma(a0, b0, k);
            load_b(b0, k + 2 * U);
            load_w(a0, k + 2 * U);
            mma(a1, b1, k + U);
            load_b(b1, k + 3 * U);
            load_w(a1, k + 3 * U);
        }
#pragma nounroll
        for (; k < kb; k += 2 * U) {
            mma(a0, b0, k);
            if (k + 2 * U < kb) {
                load_b(b0, k + 2 * U);
                load_w(a0, k + 2 * U);
            }
            mma(a1, b1, k + U);
            if (k + 3 * U < kb) {
                load_b(b1, k + 3 * U);
                load_w(a1, k + 3 * U);
            }
        }
    }
    // columns n and n + 8 hold the hi and lo products of token n; the wavefront's slots: [slot][token][16 rows]
    float *slot = (float *)(lds_raw + wave * WB);
    if (HALF) {
        // rows 0..7 of the first product and 8..15 of the second are the half tile's, each over its own k-steps: added up in the order of
        // a whole tile's sums, so that equal rows of a head have equal logits wherever they lie
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned u = __float_as_uint(gq < 2 ? acch[0][e] : acch[1][e]);
            const auto v = __builtin_amdgcn_permlane32_swap(u, u, false, false);       // the lower and the upper lanes' values, everywhere
            acch[0][e] = add_lane_xor8(__uint_as_float(v[0]) + __uint_as_float(v[1]));
        }
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[f][0][e] = add_lane_xor8(acc[f][0][e] + acc[f][1][e]);
    if (n < g.m) {
#pragma unroll
        for (int f = 0; f < NF; ++f) *(f32x4 *)(slot + f * 128 + n * 16 + gq * 4) = acc[f][0];
        if (HALF && gq < 2) *(f32x4 *)(slot + NF * 128 + n * 16 + gq * 4) = acch[0];
    }
    __syncthreads();
    if (wave >= H) return;

    const float scale = FROM_X || g.ssq_in ? inv_rms<FROM_X>(g, ssq_part, et) : 1.0f;
    const float *base = (const float *)lds_raw + et * 16 + ei;
    constexpr int WF = WB / 4;                                  // floats from one wavefront's slots to the next one's
    auto sum_rows = [&](const float *p) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kProjWaves; ++w) v += p[w * WF];
        return v;
    };
    if (g.epi == EPI_SWIGLU) {
        // rows 0..7 of a tile are gate, 8..15 up of the same features
        const int f = (full0 + wave) * 8 + ei;
        if (!HALF && wave < NF && et < g.m && f * 2 < g.N) {
            const float gate = scale * sum_rows(base + wave * 128), up = scale * sum_rows(base + wave * 128 + 8);
            store_act<F16>(g.Bnext, g.Bnext_KT, f, et, gate / (1.0f + __expf(-gate)) * up);
        }
        return;
    }
    if (g.epi != EPI_HEAD && !on) return;
    float v;
    if (HALF && (upper ? wave == 0 : wave == H - 1)) {
        v = sum_rows(base + NF * 128);
    } else {
        const int r = wave - (HALF ? upper : 0);                // half r of the whole tiles
        v = sum_rows(base + (r >> 1) * 128 + (r & 1) * 8);
    }
    v *= scale;
    if (g.epi == EPI_HEAD) {
        if (g.logits && on) g.logits[(size_t)et * g.N + row] = v;
        if (g.head_stats) {
            // (max, sum of exp, argmax) of these 8 rows, a partial of each wavefront (a maximum that started as a value that is
            // no number would keep its index and take the others' values)
            const bool num = on && v == v;
            float M = num ? v : -INFINITY, S = num ? 1.0f : on ? v : 0.f;
            int I = num ? row : 0x7fffffff;
#pragma unroll
            for (int off = 4; off > 0; off >>= 1) max_merge(M, S, I, __shfl_xor(M, off), __shfl_xor(S, off), __shfl_xor(I, off));
            if (ei == 0 && et < g.m) {
                float *o = g.head_part + ((size_t)unit * 8 + et) * 4;
                o[0] = M;
                o[1] = S;
                o[2] = __int_as_float(I);
            }
        }
    } else if (g.epi == EPI_STORE) {
        g.out[(size_t)et * g.ld + row] = v;
    } else if (g.epi == EPI_PACK) {
        store_act<F16>(g.Bnext, g.Bnext_KT, row, et, v);
    } else {
        const float y = resid + v;
        g.out[(size_t)et * g.ld + row] = y;
        if (g.Bnext) {
            // input of the next projection: y * norm weight, packed; and these 8 rows' share of sum(y^2)
            store_act<F16>(g.Bnext, g.Bnext_KT, row, et, y * next_w);
            const float q = sum8(y * y);
            if (ei == 0) g.ssq_out[(size_t)unit * 8 + et] = q;
        }
    }
}

template <int NPL, int H, int U, bool F16, bool FROM_X>
int launch_as(const GemmArgs &g, const LaunchCtx &c) {
    constexpr size_t lds = proj_lds_bytes(H, FROM_X);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_proj<NPL, H, U, F16, FROM_X>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    return launch<k_proj<NPL, H, U, F16, FROM_X>>(c, dim3((2 * g.NT + H - 1) / H), dim3(kProjThreads), lds, g.W, FROM_X ? (const void *)g.x : g.B, g.norm_w,
                                                  two(g.NT, g.KT), two(g.K, g.m), two(g.ldx, g.N), (const GemmOut &)g);
}

template <int NPL, int H, bool F16>
int launch_src(const GemmArgs &g, const LaunchCtx &c) {
    constexpr int U = proj_batch(NPL);
    if (NPL == 1 && g.KT <= kProjWaves * 2 * kProjSmallBatch)
        return g.x ? launch_as<NPL, H, kProjSmallBatch, F16, true>(g, c) : launch_as<NPL, H, kProjSmallBatch, F16, false>(g, c);
    return g.x ? launch_as<NPL, H, U, F16, true>(g, c) : launch_as<NPL, H, U, F16, false>(g, c);
}

template <int NPL, bool F16>
int launch_halves(const GemmArgs &g, int halves, const LaunchCtx &c) {
    if (halves == 2) return launch_src<NPL, 2, F16>(g, c);
    if (halves == 3) return launch_src<NPL, 3, F16>(g, c);
    return launch_src<NPL, 4, F16>(g, c);
}

}  // namespace

// what a kernel that starts from fp32 rows has: their norm weights, two batches of k-steps per wavefront at most, no residual
static bool rows_covered(const GemmArgs &g, int planes) { return g.norm_w && g.epi != EPI_RESID && g.KT <= kProjWaves * 2 * proj_batch(planes); }

bool proj_covers(const GemmArgs &g, int planes, int n_wg) {
    if (g.mode == GEMM_STREAMED) return true;
    if (g.NT > 2 * n_wg) return false;
    return !g.x || rows_covered(g, planes);
}

// halves of a row tile per workgroup: 2, 3 or 4
static int proj_halves(int n_tiles, int n_wg) {
    const int h = (2 * n_tiles + n_wg - 1) / n_wg;
    return h < 2 ? 2 : h > 3 ? 4 : h;
}

int proj_head_parts(int n_tiles, int n_wg) {
    const int h = proj_halves(n_tiles, n_wg);
    return (2 * n_tiles + h - 1) / h * h;
}

int launch_proj(const GemmArgs &g, int planes, const LaunchCtx &c) {
    if (g.x && !rows_covered(g, planes)) return (int)hipErrorInvalidValue;
    int halves = proj_halves(g.NT, c.n_wg);
    if (halves == 3 && g.epi == EPI_SWIGLU) halves = 4;
    if (planes != 1) return launch_halves<3, false>(g, halves, c);
    return g.elem == kElemF16 ? launch_halves<1, true>(g, halves, c) : launch_halves<1, false>(g, halves, c);
}

}  // namespace ad
