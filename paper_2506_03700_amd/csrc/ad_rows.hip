// Projections with many row tiles per workgroup: gate/up, the QKV projection of wide models, the exit-head transform of wide
// models, and the vocabulary pass of Eq. 1 / Eq. 2.     out[t][n] = sum_k W[n][k] * act[t][k],  m <= 8 tokens
//
// Bound by reading W once.  8 wavefronts per workgroup; wavefront w owns k-steps [KT * w / 8, KT * (w + 1) / 8) of all the
// workgroup's row tiles and keeps its part of the activations in registers (KS k-steps at most), so that only weights are
// loaded while the rows go by: two batches of U k-steps are in flight, each refilled as soon as it is multiplied; the refills
// of all tiles but the last are unconditional, so that a product waits for its own operands only.  The wavefronts' sums meet in
// LDS every 8 tiles (two sets of slots, so that one barrier per round is enough), wavefront w then finishes tile w of the round:
// what a call costs beyond the weights is a chain of instructions at its start and its end, a wavefront issues one every 5
// cycles or so, and the kernels before this one had 7000 to 10000 of them (here 1600 to 4400).  Layer step against those: 13B shape,
// 2 rows, context 777 128.0 -> 119.2 us (QKV 29.9 -> 26.0, gate/up 48.5 -> 43.9: its 20 k-steps per wavefront are two batches of
// 10 now, not 8 + 8 + 4), 8B shape, 1 row 89.9 -> 89.0, four fp16 layers 369.5 -> 358.7; exit head of 128256 tokens 185.5 -> 181.2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_launch.h"
#include "ad_proj_device.h"

namespace ad {

namespace {

constexpr int kRoundTiles = 8;              // row tiles summed together, one per wavefront
constexpr int kRoundBytes = kRoundTiles * 512;      // of a wavefront's slots: [tile][token][16 rows]
constexpr size_t kRowsLdsBytes = (size_t)2 * kProjWaves * kRoundBytes + kProjWaves * 8 * 4 + kProjWaves * 8 * 3 * 4;
static_assert(kStripBytes <= 2 * kRoundBytes, "a wavefront's strip lies in the slots");

// k-steps per batch of loads, for wavefronts of up to KS k-steps: whole numbers of batches, an even number of them per tile
constexpr int rows_batch(int npl, int ks) { return npl == 1 ? (ks == 32 ? 8 : ks / 2) : (ks == 2 ? 1 : 2); }

template <int NPL, int KS, bool F16, bool FROM_X>
__global__ void __launch_bounds__(kProjThreads, 2) k_rows(const void *weights, const void *act, const void *norm_w, uint64_t kt_k, uint64_t m_ldx, uint64_t tq_tr, GemmOut rest) {
    ProjArgs g;
    (GemmOut &)g = rest;
    g.W = weights; g.x = (const float *)act; g.B = act; g.norm_w = norm_w;
    g.KT = (int)kt_k; g.K = (int)(kt_k >> 32); g.m = (int)m_ldx; g.ldx = (int)(m_ldx >> 32); g.tq = (int)tq_tr; g.tr = (int)(tq_tr >> 32);
    const KernelArgLines<48 + sizeof(GemmOut)> lines;
    constexpr int U = rows_batch(NPL, KS), NB = KS / U, TB = NPL * 1024;
    static_assert(NB % 2 == 0 && NB * U == KS, "batches of a tile");
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, gq = lane >> 4;
    float *slots = (float *)lds_raw;                            // [2][wave][tile][token][16 rows]
    float *ssq_part = (float *)(lds_raw + 2 * kProjWaves * kRoundBytes), *best = ssq_part + kProjWaves * 8;

    const int wg = blockIdx.x, KT = g.KT;
    const int t0 = wg * g.tq + (wg < g.tr ? wg : g.tr), t1 = t0 + g.tq + (wg < g.tr ? 1 : 0);
    const int ka = (KT * wave) / kProjWaves, kb = (KT * (wave + 1)) / kProjWaves, nks = kb - ka;

    // weights: uniform base, 32-bit byte offsets (a packed matrix has less than 4 GiB)
    const char *W = (const char *)g.W;
    const unsigned tstride = (unsigned)KT * TB;
    unsigned wo = ((unsigned)t0 * (unsigned)KT + (unsigned)ka) * TB + (unsigned)lane * 16u;
    bf16x8 a[2][U][NPL];
    // batch p of the tile at byte offset o; k-steps past the wavefront's repeat its last one (products skipped)
    auto load_w = [&](bf16x8 (&d)[U][NPL], unsigned o, int p) {
        if ((p + 1) * U <= nks) {
            const char *s = W + (size_t)(o + (unsigned)(p * U * TB));
#pragma unroll
            for (int j = 0; j < U; ++j)
#pragma unroll
                for (int q = 0; q < NPL; ++q) d[j][q] = load_weights(s + j * TB + q * 1024);
        } else {
            const int ok = nks > 0 ? nks - 1 : 0;               // (ka < KT also without any k-steps)
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int jj = p * U + j < ok ? p * U + j : ok;
#pragma unroll
                for (int q = 0; q < NPL; ++q) d[j][q] = load_weights(W + (size_t)(o + (unsigned)(jj * TB)) + q * 1024);
            }
        }
    };
    bf16x8 b[KS];
    auto first_weights = [&]() {
        load_w(a[0], wo, 0);
        load_w(a[1], wo, 1);
        lines.use();
    };
    if constexpr (FROM_X) {
        operand_from_rows<NPL, KS, F16>(g, ka, kb, lane, (uint16_t *)(lds_raw + wave * 2 * kRoundBytes), ssq_part + wave * 8, first_weights,
                                        [&](int j, bf16x8 v) { b[j] = v; });
        __syncthreads();                                        // the strips lie in other wavefronts' slots
    } else {
        // lanes of tokens past the call's read token 0's operands (the same cache lines), k-steps past the wavefront's some valid one
        const unsigned bo = (unsigned)((n & 7) < g.m ? (n & 7) : 0) * (unsigned)KT * 128u + (unsigned)((n >> 3) * 64 + gq * 16);
        const char *B = (const char *)g.B;
        if (nks == KS) {
            const char *s = B + (size_t)(bo + (unsigned)ka * 128u);
#pragma unroll
            for (int j = 0; j < KS; ++j) b[j] = *(const bf16x8 *)(s + j * 128);
        } else {
            const int ok = nks > 0 ? kb - 1 : ka;
#pragma unroll
            for (int j = 0; j < KS; ++j) b[j] = *(const bf16x8 *)(B + (bo + (unsigned)(ka + j < ok ? ka + j : ok) * 128u));
        }
        float sq[8];
        if (g.ssq_in && wave < g.m) {
            // the first 512 partial sums of squares are requested ahead of the weights
#pragma unroll
            for (int i = 0; i < 8; ++i) sq[i] = g.ssq_in[(size_t)(lane + 64 * i < g.ssq_tiles ? lane + 64 * i : 0) * 8 + wave];
        }
        first_weights();
        if (g.ssq_in && wave < g.m) {
            float v = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) v += lane + 64 * i < g.ssq_tiles ? sq[i] : 0.f;
            for (int i = lane + 512; i < g.ssq_tiles; i += 64) v += g.ssq_in[(size_t)i * 8 + wave];
            v = sum64(v);
            if (lane == 0) ssq_part[wave] = v;
        }
    }

    // lane = token * 8 + row of the tile's lower half: two outputs each
    const int et = lane >> 3, ei = lane & 7;
    float scale = 1.0f;
    bool scale_set = false;
    float best_m = -INFINITY, best_s = 0.f;                     // EPI_HEAD: (max, sum of exp, argmax) of this lane's rows
    int best_i = 0x7fffffff;
    // tiles [ta, ta + nt) are in slot set `set`
    auto finish = [&](int set, int ta, int nt) {
        __syncthreads();
        if (!scale_set) {
            scale_set = true;
            if (FROM_X || g.ssq_in) scale = inv_rms<FROM_X>(g, ssq_part, et);
        }
        if (wave >= nt || et >= g.m) return;
        const float *s = slots + (size_t)set * kProjWaves * (kRoundBytes / 4) + wave * 128 + et * 16 + ei;
        float v0 = 0.f, v1 = 0.f;
#pragma unroll
        for (int w = 0; w < kProjWaves; ++w) {
            v0 += s[w * (kRoundBytes / 4)];
            v1 += s[w * (kRoundBytes / 4) + 8];
        }
        v0 *= scale;
        v1 *= scale;
        const int tile = ta + wave, row = tile * 16 + ei;
        if (g.epi == EPI_SWIGLU) {
            // rows 0..7 of a tile are gate, 8..15 up of the same features
            if (row < g.N) store_act<F16>(g.Bnext, g.Bnext_KT, tile * 8 + ei, et, v0 / (1.0f + __expf(-v0)) * v1);
        } else if (g.epi == EPI_STORE) {
            float *o = g.out + (size_t)et * g.ld + row;
            if (row < g.N) o[0] = v0;
            if (row + 8 < g.N) o[8] = v1;
        } else if (g.epi == EPI_PACK) {
            if (row < g.N) store_act<F16>(g.Bnext, g.Bnext_KT, row, et, v0);
            if (row + 8 < g.N) store_act<F16>(g.Bnext, g.Bnext_KT, row + 8, et, v1);
        } else {
            if (g.logits) {
                float *o = g.logits + (size_t)et * g.N + row;
                if (row < g.N) o[0] = v0;
                if (row + 8 < g.N) o[8] = v1;
            }
            if (g.head_stats) {
                if (row < g.N) max_merge(best_m, best_s, best_i, v0, 1.0f, row);
                if (row + 8 < g.N) max_merge(best_m, best_s, best_i, v1, 1.0f, row + 8);
            }
        }
    };

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const bf16x8 (&w)[U][NPL], int p) {
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (p * U + j < nks) {
#pragma unroll
                for (int q = 0; q < NPL; ++q) acc = mma16<F16>(w[j][q], b[p * U + j], acc);
            }
    };
    int slot = 0, set = 0;
    // columns n and n + 8 hold the hi and lo products of token n
    auto end_tile = [&]() {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = add_lane_xor8(acc[e]);
        if (n < g.m) *(f32x4 *)(slots + (size_t)(set * kProjWaves + wave) * (kRoundBytes / 4) + slot * 128 + n * 16 + gq * 4) = acc;
        acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        ++slot;
    };
    int t = t0;
#pragma nounroll
    for (; t + 1 < t1; ++t) {
#pragma unroll
        for (int p = 0; p < NB; ++p) {
            mma(a[p & 1], p);
            if (p + 2 < NB) load_w(a[p & 1], wo, p + 2);
            else load_w(a[p & 1], wo + tstride, p + 2 - NB);
        }
        wo += tstride;
        end_tile();
        if (slot == kRoundTiles) {
            finish(set, t + 1 - kRoundTiles, kRoundTiles);
            slot = 0;
            set ^= 1;
        }
    }
#pragma unroll
    for (int p = 0; p < NB; ++p) {
        mma(a[p & 1], p);
        if (p + 2 < NB) load_w(a[p & 1], wo, p + 2);
    }
    end_tile();
    finish(set, t1 - slot, slot);

    if (g.epi == EPI_HEAD && g.head_stats) {
        // per token: over the 8 lanes, then over the wavefronts, which the partials' reader folds in workgroup order
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) max_merge(best_m, best_s, best_i, __shfl_xor(best_m, off), __shfl_xor(best_s, off), __shfl_xor(best_i, off));
        float *p = best + (wave * 8 + et) * 3;
        if (ei == 0) {
            p[0] = best_m;
            p[1] = best_s;
            p[2] = __int_as_float(best_i);
        }
        __syncthreads();
        if (tid < g.m) {
            float M = -INFINITY, S = 0.f;
            int I = 0x7fffffff;
#pragma unroll
            for (int w = 0; w < kProjWaves; ++w) {
                const float *q = best + (w * 8 + tid) * 3;
                max_merge(M, S, I, q[0], q[1], __float_as_int(q[2]));
            }
            float *o = g.head_part + ((size_t)wg * 8 + tid) * 4;
            o[0] = M;
            o[1] = S;
            o[2] = __int_as_float(I);
        }
    }
}

template <int NPL, int KS, bool F16, bool FROM_X>
int launch_as(const GemmArgs &g, int grid, const LaunchCtx &c) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_rows<NPL, KS, F16, FROM_X>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRowsLdsBytes);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    GemmArgs ga = g;
    set_tile_partition(ga, grid);
    return launch<k_rows<NPL, KS, F16, FROM_X>>(c, dim3(grid), dim3(kProjThreads), kRowsLdsBytes, ga.W, FROM_X ? (const void *)ga.x : ga.B, ga.norm_w,
                                                two(ga.KT, ga.K), two(ga.m, ga.ldx), two(ga.tq, ga.tr), (const GemmOut &)ga);
}

template <int NPL, int KS, bool F16>
int launch_src(const GemmArgs &g, int grid, const LaunchCtx &c) {
    return g.x ? launch_as<NPL, KS, F16, true>(g, grid, c) : launch_as<NPL, KS, F16, false>(g, grid, c);
}

// The instance whose registers hold the activations of a wavefront: 16-bit models of d_model <= 512, 1024, 2048, 4096, 5120, 6144, 8192.  An
// instance goes through its k-steps whether a wavefront has them or not (loads of its last one again, no products): with 8 as the fewest an
// exit head of 128256 tokens took 56.9 us at d_model 512 and 55.6 at 1024, 27.6 and 42.4 with 2 and 4 (54.5 and 61.3 with the kernel before
// this one).
template <bool F16>
int launch16(const GemmArgs &g, int nks, int grid, const LaunchCtx &c) {
    if (nks <= 2) return launch_src<1, 2, F16>(g, grid, c);
    if (nks <= 4) return launch_src<1, 4, F16>(g, grid, c);
    if (nks <= 8) return launch_src<1, 8, F16>(g, grid, c);
    if (nks <= 16) return launch_src<1, 16, F16>(g, grid, c);
    if (nks <= 20) return launch_src<1, 20, F16>(g, grid, c);
    if (nks <= 24) return launch_src<1, 24, F16>(g, grid, c);
    return launch_src<1, 32, F16>(g, grid, c);
}

// the same for fp32 models of d_model <= 512, 1024, 2048, 3072, 4096, 5120: with 2 and 20 k-steps alone the logits of 32016 tokens took
// 68.6 us at d_model 1024 and 86.0 at 2048, 31.0 and 61.3 with these (and 35.0 and 66.5 with the kernel before this one)
int launch32(const GemmArgs &g, int nks, int grid, const LaunchCtx &c) {
    if (nks <= 2) return launch_src<3, 2, false>(g, grid, c);
    if (nks <= 4) return launch_src<3, 4, false>(g, grid, c);
    if (nks <= 8) return launch_src<3, 8, false>(g, grid, c);
    if (nks <= 12) return launch_src<3, 12, false>(g, grid, c);
    if (nks <= 16) return launch_src<3, 16, false>(g, grid, c);
    return launch_src<3, 20, false>(g, grid, c);
}

}  // namespace

int rows_max_k(int planes) { return (planes == 1 ? 32 : 20) * kProjWaves * 32; }

int launch_rows(const GemmArgs &g, int planes, int grid, const LaunchCtx &c) {
    if (g.KT * 32 > rows_max_k(planes) || g.K < 8 || (g.x && !g.norm_w) || g.epi == EPI_RESID) return (int)hipErrorInvalidValue;
    const int nks = (g.KT + kProjWaves - 1) / kProjWaves;       // most k-steps of a wavefront
    if (planes != 1) return launch32(g, nks, grid, c);
    return g.elem == kElemF16 ? launch16<true>(g, nks, grid, c) : launch16<false>(g, nks, grid, c);
}

}  // namespace ad
