// Sampled decoding (Sec. 2.2 of arxiv 2506.03700): the token of Eq. 1 drawn from softmax(z / T), and the
// verification of Eq. 2 in its general form -- a drafted token t survives with probability
// min(1, p*(t) / p_draft(t)); the first rejected draft is replaced by a draw from
// Normalize(max(0, p* - p_draft)); if none is rejected the next token is drawn from the newest row's p*.
//
// Every draw is a uniform number u in [0, 1) handed in by the caller and turned into a token by inversion of
// the cumulative distribution in token-id order: the first id whose cumulative weight exceeds u * (total
// weight).  A row is cut into segments of consecutive ids, one workgroup each: a first kernel leaves each segment's maximum
// and sum of weights, a second one (one workgroup) finds the segment that holds the target from those and walks that
// segment alone.  What bounds these calls is not the row (0.5 MB) but the chain of dependent loads, reductions and kernel
// boundaries: with one workgroup that passed over the whole row three times a draw from 128256 logits took 97 us on the
// GPU; the sums are added up in a fixed order (no float atomics), so everything is deterministic.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ad_internal.h"

namespace ad {

namespace {

constexpr int kSampleThreads = 256;
constexpr int kSampleWaves = kSampleThreads / 64;
constexpr int kSegIds = 2048;                    // ids per segment, until there are as many segments as a workgroup has threads

struct SampleLds {
    float wave_val[kSampleWaves];
    float bcast[4];
    int best;
    int last_pos;
};

// (largest value, sum of the weights relative to it) of a segment
struct SegStat { float mx, sum; };

__device__ __forceinline__ float wave_max(float v) {
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

// max over the workgroup, returned to every thread
__device__ __forceinline__ float block_max(float v, SampleLds &L) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) L.wave_val[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = L.wave_val[0];
#pragma unroll
    for (int w = 1; w < kSampleWaves; ++w) r = fmaxf(r, L.wave_val[w]);
    return r;
}

// Exclusive prefix of `local` over the threads in thread order (fixed association: butterfly-free scan inside a
// wavefront, then the wavefront totals in order); *total receives the sum over the workgroup.
__device__ __forceinline__ float block_exclusive_scan(float local, SampleLds &L, float *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float incl = local;
    for (int off = 1; off < 64; off <<= 1) {
        const float up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    __syncthreads();
    if (lane == 63) L.wave_val[wave] = incl;
    __syncthreads();
    float before = 0.f, all = 0.f;
#pragma unroll
    for (int w = 0; w < kSampleWaves; ++w) {
        if (w < wave) before += L.wave_val[w];
        all += L.wave_val[w];
    }
    *total = all;
    return before + (incl - local);
}

// a segment's sum relative to the row's largest value (a segment without weight has none, whatever its maximum)
__device__ __forceinline__ float rescaled(SegStat s, float mx, float inv_t) {
    return (s.sum == 0.f) ? 0.f : s.sum * expf((s.mx - mx) * inv_t);
}

// Inversion draw over the weights w(j) >= 0 of a row whose segments' statistics are in `seg` (thread t: segment t; the
// weights are relative to mx, a segment's to its own maximum, which inv_t scales).  Returns (to every thread) the token, its
// weight and the total weight.  No id of positive weight: token -1.
template <class W>
__device__ __forceinline__ int sample_segments(W w, const SegStat *seg, float mx, float inv_t, int V, int n_seg, int seg_ids, float u, SampleLds &L,
                                               float *w_tok, float *total_out) {
    const int tid = threadIdx.x;
    const float mine = tid < n_seg ? rescaled(seg[tid], mx, inv_t) : 0.f;
    float total;
    const float before = block_exclusive_scan(mine, L, &total);
    if (tid == 0) {
        L.best = 0x7fffffff;
        L.last_pos = -1;
    }
    __syncthreads();
    const float target = u * total;
    if (mine > 0.f && before + mine > target) atomicMin(&L.best, tid);
    __syncthreads();
    const int s = L.best;
    if (s != 0x7fffffff && tid == s) L.bcast[1] = before;
    __syncthreads();
    int tok = -1;
    if (s != 0x7fffffff) {
        // walk the segment: thread t owns consecutive ids, added up in id order
        const int per = (seg_ids + kSampleThreads - 1) / kSampleThreads;
        const int end = min(V, (s + 1) * seg_ids), j0 = min(end, s * seg_ids + tid * per), j1 = min(end, j0 + per);
        float local = 0.f;
        int last = -1;
        for (int j = j0; j < j1; ++j) {
            const float x = w(j);
            local += x;
            if (x > 0.f) last = j;
        }
        float seg_total;
        const float at = L.bcast[1] + block_exclusive_scan(local, L, &seg_total);
        if (tid == 0) L.best = 0x7fffffff;
        __syncthreads();
        if (at + local > target || at > target) {
            float c = at;
            for (int j = j0; j < j1; ++j) {
                const float x = w(j);
                c += x;
                if (c > target && x > 0.f) {
                    atomicMin(&L.best, j);
                    break;
                }
            }
        }
        if (last >= 0) atomicMax(&L.last_pos, last);
        __syncthreads();
        // the two ways of adding the segment up may round differently: then its last id of positive weight
        tok = (L.best != 0x7fffffff) ? L.best : L.last_pos;
    }
    if (tok < 0) {
        // rounding left nothing above the target (u * total == total), or a sum is not a number: the row's last id of
        // positive weight
        __syncthreads();
        int last = -1;
        for (int j = tid; j < V; j += kSampleThreads)
            if (w(j) > 0.f) last = j;
        if (tid == 0) L.last_pos = -1;
        __syncthreads();
        if (last >= 0) atomicMax(&L.last_pos, last);
        __syncthreads();
        tok = L.last_pos;
    }
    *w_tok = tok >= 0 ? w(tok) : 0.f;
    *total_out = total;
    return tok;
}

struct SoftmaxWeight {
    const float *z; float mx, inv_t;
    __device__ __forceinline__ float operator()(int j) const { return expf((z[j] - mx) * inv_t); }
};

// max(0, p*(j) - p_draft(j)) up to a common factor, from the log-probabilities a = log p*(j), b = log p_draft(j):
// exp(a - c) * (1 - exp(b - a)) where a > b, with c = the largest such a.  Working relative to c keeps the weights
// in range when every token on which p* exceeds p_draft has a probability far below the smallest fp32 number
// (a dominant token that both distributions agree on leaves exactly that), and 1 - exp(b - a) through expm1 keeps
// the difference of two nearly equal probabilities accurate.
struct ResidualWeight {
    const float *zf, *zq; float mf, lsf, mq, lsq, inv_t, c;
    __device__ __forceinline__ float log_p(int j) const { return (zf[j] - mf) * inv_t - lsf; }
    __device__ __forceinline__ float log_q(int j) const { return (zq[j] - mq) * inv_t - lsq; }
    __device__ __forceinline__ float operator()(int j) const {
        const float a = log_p(j), b = log_q(j);
        return a > b ? expf(a - c) * -expm1f(b - a) : 0.f;
    }
};

// Statistics of segment blockIdx.x of row blockIdx.y: rows [0, n_first) start at z0, the others at z1.
struct SegArgs { const float *z0, *z1; int n_first, V, n_seg, seg_ids; float inv_t; SegStat *out; };

__global__ void __launch_bounds__(kSampleThreads) k_segment_stats(SegArgs a) {
    __shared__ SampleLds L;
    const int r = blockIdx.y, tid = threadIdx.x;
    const float *z = r < a.n_first ? a.z0 + (size_t)r * a.V : a.z1 + (size_t)(r - a.n_first) * a.V;
    const int j0 = blockIdx.x * a.seg_ids, j1 = min(a.V, j0 + a.seg_ids);
    float m = -INFINITY;
    for (int j = j0 + tid; j < j1; j += kSampleThreads) m = fmaxf(m, z[j]);
    m = block_max(m, L);
    float s = 0.f;
    if (m != -INFINITY)
        for (int j = j0 + tid; j < j1; j += kSampleThreads) s += expf((z[j] - m) * a.inv_t);
    float total;
    (void)block_exclusive_scan(s, L, &total);
    if (tid == 0) a.out[(size_t)r * a.n_seg + blockIdx.x] = SegStat{m, total};
}

// (max z, sum exp((z - max) * inv_t)) of a row from its segments, by one wavefront, to all its lanes
__device__ __forceinline__ SegStat row_from_segments(const SegStat *seg, int n_seg, float inv_t) {
    const int lane = threadIdx.x & 63;
    SegStat v[kSampleThreads / 64];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kSampleThreads / 64; ++i) {
        v[i] = lane + 64 * i < n_seg ? seg[lane + 64 * i] : SegStat{-INFINITY, 0.f};
        m = fmaxf(m, v[i].mx);
    }
    m = wave_max(m);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < kSampleThreads / 64; ++i) s += rescaled(v[i], m, inv_t);
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    return SegStat{m, s};
}

__global__ void __launch_bounds__(kSampleThreads) k_sample_row(SampleArgs a, const SegStat *seg, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    const float mx = block_max((int)threadIdx.x < n_seg ? seg[threadIdx.x].mx : -INFINITY, L);
    float w_tok, total;
    const int tok = sample_segments(SoftmaxWeight{a.z, mx, a.inv_t}, seg, mx, a.inv_t, a.V, n_seg, seg_ids, a.u, L, &w_tok, &total);
    if (threadIdx.x == 0) {
        *a.tok_out = tok;
        *a.prob_out = w_tok / total;
    }
}

// Eq. 2 over the drafts, computed by every workgroup that needs the outcome (the same sums in the same order).
struct Decision { int n_acc, rejected; SegStat f, q; };      // of row n_acc: statistics of its final and draft logits

__device__ __forceinline__ Decision decide(const VerifySampledArgs &a, const SegStat *seg, int n_seg, bool write_ratio) {
    __shared__ SegStat row[15];
    __shared__ int s_nacc, s_rejected;
    const int wave = threadIdx.x >> 6, n_draft = a.m - 1;
    for (int r = wave; r < 2 * a.m - 1; r += kSampleWaves) {
        const SegStat st = row_from_segments(seg + (size_t)r * n_seg, n_seg, a.inv_t);
        if ((threadIdx.x & 63) == 0) row[r] = st;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int nacc = n_draft, rejected = 0;
        for (int k = 0; k < n_draft; ++k) {
            float ratio = 0.f;
            if (!rejected) {
                const int t = a.draft[k];
                // p*(t) / p_draft(t) through the logarithms, so that two tiny probabilities still have a ratio
                const float lp = (a.zf[(size_t)k * a.V + t] - row[k].mx) * a.inv_t - logf(row[k].sum);
                const float lq = (a.zq[(size_t)k * a.V + t] - row[a.m + k].mx) * a.inv_t - logf(row[a.m + k].sum);
                ratio = expf(lp - lq);
                if (!(a.u_accept[k] < fminf(1.0f, ratio))) {
                    rejected = 1;
                    nacc = k;
                }
            }
            if (write_ratio && a.ratio_out) a.ratio_out[k] = ratio;
        }
        s_nacc = nacc;
        s_rejected = rejected;
    }
    __syncthreads();
    Decision d;
    d.n_acc = s_nacc;
    d.rejected = s_rejected;
    d.f = row[d.n_acc];
    d.q = d.rejected ? row[a.m + d.n_acc] : SegStat{0.f, 0.f};
    return d;
}

__device__ __forceinline__ ResidualWeight residual_of(const VerifySampledArgs &a, const Decision &d) {
    return ResidualWeight{a.zf + (size_t)d.n_acc * a.V, a.zq + (size_t)d.n_acc * a.V, d.f.mx, logf(d.f.sum), d.q.mx, logf(d.q.sum), a.inv_t, 0.f};
}

// The residual's segments if a draft was rejected: (largest log p* where p* exceeds p_draft, sum of the weights relative to it).
__global__ void __launch_bounds__(kSampleThreads) k_residual_segments(VerifySampledArgs a, const SegStat *seg, int n_seg, int seg_ids, SegStat *out) {
    __shared__ SampleLds L;
    const Decision d = decide(a, seg, n_seg, false);
    if (!d.rejected) return;
    ResidualWeight w = residual_of(a, d);
    const int j0 = blockIdx.x * seg_ids, j1 = min(a.V, j0 + seg_ids);
    float c = -INFINITY;
    for (int j = j0 + threadIdx.x; j < j1; j += kSampleThreads) {
        const float la = w.log_p(j);
        if (la > w.log_q(j)) c = fmaxf(c, la);
    }
    w.c = block_max(c, L);
    float s = 0.f;
    if (w.c != -INFINITY)
        for (int j = j0 + threadIdx.x; j < j1; j += kSampleThreads) s += w(j);
    float total;
    (void)block_exclusive_scan(s, L, &total);
    if (threadIdx.x == 0) out[blockIdx.x] = SegStat{w.c, total};
}

__global__ void __launch_bounds__(kSampleThreads) k_verify_sampled(VerifySampledArgs a, const SegStat *seg, const SegStat *res_seg, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    const Decision d = decide(a, seg, n_seg, true);
    const int r = d.n_acc;
    int tok = -1;
    float w_tok, total;
    if (d.rejected) {
        ResidualWeight w = residual_of(a, d);
        w.c = block_max((int)threadIdx.x < n_seg ? res_seg[threadIdx.x].mx : -INFINITY, L);
        if (w.c != -INFINITY) tok = sample_segments(w, res_seg, w.c, 1.0f, a.V, n_seg, seg_ids, a.u_resample[r], L, &w_tok, &total);
        __syncthreads();
    }
    if (tok < 0)       // nothing rejected (or a residual that is identically zero): draw from the row's final distribution
        tok = sample_segments(SoftmaxWeight{a.zf + (size_t)r * a.V, d.f.mx, a.inv_t}, seg + (size_t)r * n_seg, d.f.mx, a.inv_t, a.V, n_seg, seg_ids,
                              d.rejected ? a.u_resample[r] : a.u_final, L, &w_tok, &total);
    if (threadIdx.x == 0) {
        *a.n_accept_out = r;
        *a.next_out = tok;
    }
}

// A row's segments: kSegIds ids each, and no more segments than a workgroup has threads.
void segments(int V, int *n_seg, int *seg_ids) {
    const int n = (V + kSegIds - 1) / kSegIds, most = n < kSampleThreads ? n : kSampleThreads;
    *seg_ids = (V + most - 1) / most;
    *n_seg = (V + *seg_ids - 1) / *seg_ids;
}

}  // namespace

static_assert(sizeof(SegStat) * 16 * kSampleThreads <= kSampleScratchBytes, "the segments of 15 rows and of a residual");

int launch_sample_row(const SampleArgs &a, void *stream) {
    if (a.V < 1 || !(a.inv_t > 0.f)) return (int)hipErrorInvalidValue;
    int n_seg, seg_ids;
    segments(a.V, &n_seg, &seg_ids);
    SegStat *seg = (SegStat *)a.scratch;
    hipLaunchKernelGGL(k_segment_stats, dim3(n_seg, 1), dim3(kSampleThreads), 0, (hipStream_t)stream,
                       SegArgs{a.z, nullptr, 1, a.V, n_seg, seg_ids, a.inv_t, seg});
    const int rc = (int)hipGetLastError();
    if (rc) return rc;
    hipLaunchKernelGGL(k_sample_row, dim3(1), dim3(kSampleThreads), 0, (hipStream_t)stream, a, seg, n_seg, seg_ids);
    return (int)hipGetLastError();
}

int launch_verify_sampled(const VerifySampledArgs &a, void *stream) {
    if (a.V < 1 || a.m < 1 || a.m > 8 || !(a.inv_t > 0.f)) return (int)hipErrorInvalidValue;
    for (int k = 0; k + 1 < a.m; ++k)
        if (a.draft[k] < 0 || a.draft[k] >= a.V) return (int)hipErrorInvalidValue;
    int n_seg, seg_ids;
    segments(a.V, &n_seg, &seg_ids);
    SegStat *seg = (SegStat *)a.scratch, *res_seg = seg + (size_t)(2 * a.m - 1) * n_seg;
    const dim3 wg(kSampleThreads);
    hipLaunchKernelGGL(k_segment_stats, dim3(n_seg, 2 * a.m - 1), wg, 0, (hipStream_t)stream, SegArgs{a.zf, a.zq, a.m, a.V, n_seg, seg_ids, a.inv_t, seg});
    int rc = (int)hipGetLastError();
    if (rc) return rc;
    if (a.m > 1) {
        hipLaunchKernelGGL(k_residual_segments, dim3(n_seg), wg, 0, (hipStream_t)stream, a, seg, n_seg, seg_ids, res_seg);
        if ((rc = (int)hipGetLastError())) return rc;
    }
    hipLaunchKernelGGL(k_verify_sampled, dim3(1), wg, 0, (hipStream_t)stream, a, seg, res_seg, n_seg, seg_ids);
    return (int)hipGetLastError();
}

}  // namespace ad
