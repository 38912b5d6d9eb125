// Stand-alone launches of the projections, when the layer step runs as separate kernels, and of the LM head of Eq. 1 / Eq. 2: which
// kernel (ad_proj.hip: few row tiles per workgroup, ad_rows.hip: many), and the second pass of the vocabulary reduction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_launch.h"

namespace ad {

// Second pass of the vocabulary reduction: fold the per-workgroup (max, sum of exp, argmax) partials in a
// fixed order (the lowest token id wins ties), one wavefront per token, then apply the
// verification rule of Eq. 2 at temperature 0 if asked.
__global__ void __launch_bounds__(512) k_head_combine(GemmArgs g) {
    __shared__ int idx_sh[8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave < g.m) {
        const int t = wave;
        float M = -INFINITY, S = 0.f;
        int I = 0x7fffffff;
        const f32x4 *part = (const f32x4 *)g.head_part + t;
        for (int w0 = 0; w0 < g.n_parts; w0 += 256) {           // four partials per lane are in flight
            f32x4 p[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int w = w0 + i * 64 + lane;
                p[i] = part[(size_t)(w < g.n_parts ? w : 0) * 8];
                if (w >= g.n_parts) p[i] = (f32x4){-INFINITY, 0.f, __int_as_float(0x7fffffff), 0.f};
            }
            float m = M;
#pragma unroll
            for (int i = 0; i < 4; ++i) m = fmaxf(m, p[i][0]);
            const float ref = softmax_ref(m);
            S *= __expf(M - ref);
            if (m > M) I = 0x7fffffff;
            M = m;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                S += p[i][1] * __expf(p[i][0] - ref);
                const int id = __float_as_int(p[i][2]);
                if (p[i][0] == m && id < I) I = id;
            }
        }
        const float m = max64(M), ref = softmax_ref(m);
        S = sum64(S * __expf(M - ref));
        I = min64(M == m ? I : 0x7fffffff);
        if (lane == 0) {
            idx_sh[t] = I;
            if (g.tok_out) report(g.tok_out + t, I);
            if (g.conf_out) report(g.conf_out + t, 1.0f / S);   // exp(max - logsumexp)
        }
    }
    if (g.done_flag) reported();
    __syncthreads();
    if (g.verify && threadIdx.x == 0) {
        // the first row whose final-layer token differs from the token drafted after it ends the accepted
        // run and supplies the replacement
        int acc = g.m - 1;
        for (int j = 0; j < g.m - 1; ++j)
            if (idx_sh[j] != g.draft[j]) { acc = j; break; }
        report(g.n_accept_out, acc);
        report(g.next_out, idx_sh[acc]);
    }
    if (threadIdx.x == 0) report_done(g.done_flag, g.done_seq);
}

int launch_gemm(const GemmArgs &g, int planes, const LaunchCtx &c) {
    // equal numbers of row tiles per workgroup: with per = ceil(NT / n_wg) tiles each, ceil(NT / per) workgroups
    const int grid = head_grid(g.NT, c.n_wg);
    if ((planes == 1) != (g.elem != kElemF32)) return (int)hipErrorInvalidValue;     // fp32 weights are three bf16 planes
    GemmArgs h = g;
    h.head_stats = g.epi == EPI_HEAD && (g.tok_out || g.conf_out || g.verify || g.done_flag);       // (the logits alone need no reduction)
    const bool few = proj_covers(g, planes, c.n_wg);
    int rc = few ? launch_proj(h, planes, c) : launch_rows(h, planes, grid, c);
    if (rc) return rc;
    if (h.head_stats) {
        h.n_parts = few ? proj_head_parts(g.NT, c.n_wg) : grid;
        rc = launch<k_head_combine>(c, dim3(1), dim3(512), 0, h);
    }
    return rc;
}

// ---- scratch for callers that cannot allocate --------------------------------------------------------------
// The vocabulary pass leaves one (max, sum of exp, argmax) partial per workgroup and token, which its second kernel
// folds.  Normally they live in the model's workspace; the allocation-free entry point keeps them in this
// file-scope array instead: kStaticHeadParts workgroups x 8 tokens x 4 floats = 512 KiB, held by every GPU the
// library runs on until the process ends.  In host code the array's name is only a stand-in for the symbol: its
// device address is asked for once per device (with that device current) and kept.
static __device__ __align__(256) float scratch[(size_t)kStaticHeadParts * 8 * 4];

int static_head_scratch(float **ptr) {
    constexpr int kMaxDevices = 64;
    static float *addr[kMaxDevices];
    static bool have[kMaxDevices];
    static std::mutex mu;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!have[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        addr[dev] = (float *)p;
        have[dev] = true;
    }
    *ptr = addr[dev];
    return 0;
}

int head_parts(int n_tiles, int n_wg) {
    const int a = head_grid(n_tiles, n_wg), b = n_tiles <= 2 * n_wg ? proj_head_parts(n_tiles, n_wg) : 0;
    return a > b ? a : b;
}

int head_grid(int n_tiles, int n_wg) {
    const int per = (n_tiles + n_wg - 1) / n_wg;
    const int grid = (n_tiles + per - 1) / (per < 1 ? 1 : per);
    return grid < 1 ? 1 : grid;
}

}  // namespace ad
