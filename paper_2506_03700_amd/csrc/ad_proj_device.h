// Device code shared by the kernels of the layer step's projections (ad_proj.hip: few row tiles per workgroup, ad_rows.hip: many).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ad_device.h"
#include "ad_internal.h"

namespace ad {

constexpr int kProjWaves = 8;
constexpr int kProjThreads = kProjWaves * 64;
constexpr int kStripBytes = 8192;            // a wavefront's 8 k-steps of activations, in operand order

__device__ __forceinline__ bf16x8 load_weights(const char *p) { return __builtin_nontemporal_load((const bf16x8 *)p); }

// The B operand of this wavefront's k-steps [ka, kb), at most KS of them, from fp32 rows: put(j, v) receives the operand registers of
// k-step ka + j.  Passes of 8 k-steps = 256 inputs: lane l takes inputs 4l .. 4l+3 of every token, multiplies by the norm weights,
// splits and writes them in operand order into its wavefront's strip of LDS, from which each lane reads its operand registers.
// Units of 16 bytes are permuted (u -> u ^ ((u >> 4) & 15)) so that the 8-byte writes of a wavefront, which all go to the same
// operand column, spread over the LDS banks.  Columns of tokens past the call's hold whatever the strip held.  The rows of two
// passes are requested first, then `weights` puts the first weights in flight.  ssq_part[t] receives the sum of squares of
// token t's inputs here.
template <int NPL, int KS, bool F16, class Weights, class Put>
__device__ __forceinline__ void operand_from_rows(const ProjArgs &g, int ka, int kb, int lane, uint16_t *strip16, float *ssq_part, Weights weights, Put put) {
    constexpr int NP = (KS + 7) / 8, NX = NP < 2 ? 1 : 2;
    f32x4 xr[NX][8], wn;
    u16x4 wr[NX];
    f32x4 wf[NX];
    auto load = [&](int p) {
        const int k = (ka + p * 8) * 32 + lane * 4, kc = k < g.K - 4 ? k : g.K - 4;
        if (NPL == 3) wf[p % NX] = *(const f32x4 *)((const float *)g.norm_w + kc);
        else wr[p % NX] = *(const u16x4 *)((const uint16_t *)g.norm_w + kc);
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (t < g.m) xr[p % NX][t] = *(const f32x4 *)(g.x + (size_t)t * g.ldx + kc);
    };
#pragma unroll
    for (int p = 0; p < NX; ++p) load(p);
    weights();
    const bf16x8 *strip = (const bf16x8 *)strip16;
    auto sw = [](int u) { return u ^ ((u >> 4) & 15); };
    float ssq[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (NPL == 3) {
            wn = wf[p % NX];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) wn[e] = from16<F16>(wr[p % NX][e]);
        }
        const int ks = ka + p * 8 + (lane >> 3), k = ks * 32 + (lane & 7) * 4;
        const bool k_on = ks < kb && k < g.K;
        const int uu = (lane >> 3) * 64 + ((lane & 7) >> 1) * 16;    // unit of column 0
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (t < g.m) {
                u16x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float xv = k_on ? xr[p % NX][t][e] : 0.f;
                    ssq[t] += xv * xv;
                    uint16_t h, l;
                    split16<F16>(xv * wn[e], h, l);
                    hi[e] = h;
                    lo[e] = l;
                }
                *(u16x4 *)(strip16 + sw(uu + t) * 8 + (lane & 1) * 4) = hi;
                *(u16x4 *)(strip16 + sw(uu + 8 + t) * 8 + (lane & 1) * 4) = lo;
            }
        if (p + NX < NP) load(p + NX);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            if (p * 8 + jj < KS) put(p * 8 + jj, strip[sw(jj * 64 + lane)]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t < g.m) {
            const float v = sum64(ssq[t]);
            if (lane == 0) ssq_part[t] = v;
        }
}

// 1 / rms of token t from its sums of squares: FROM_X the wavefronts' (ssq_part[wave * 8 + t]), else the producer's (ssq_part[t])
template <bool FROM_X>
__device__ __forceinline__ float inv_rms(const ProjArgs &g, const float *ssq_part, int t) {
    float s = 0.f;
    if (FROM_X) {
#pragma unroll
        for (int w = 0; w < kProjWaves; ++w) s += ssq_part[w * 8 + t];
    } else {
        s = ssq_part[t];
    }
    return 1.0f / sqrtf(s * g.inv_dim + g.eps);
}

// Wavefront t adds up the producer's partial sums of squares of token t, per lane and then over the lanes (fixed order).
__device__ __forceinline__ void sum_ssq(const ProjArgs &g, int wave, int lane, float *ssq_part) {
    if (wave >= g.m) return;
    float v = 0.f;
    for (int i = lane; i < g.ssq_tiles; i += 64) v += g.ssq_in[(size_t)i * 8 + wave];
    v = sum64(v);
    if (lane == 0) ssq_part[wave] = v;
}

}  // namespace ad
