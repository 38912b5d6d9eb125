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

constexpr int kSampleThreads = 512;              // measured against 256 and 1024: 8 rows of 128256 logits 46.7, 51.8, 51.3 us a call
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
    float total, target;
    int s = 0;
    if (tid == 0) {
        L.best = 0x7fffffff;
        L.last_pos = -1;
        L.bcast[1] = 0.f;
    }
    if (n_seg == 1) {
        total = rescaled(seg[0], mx, inv_t);
        target = u * total;
        if (!(total > target)) s = 0x7fffffff;
        __syncthreads();
    } else {
        const float mine = tid < n_seg ? rescaled(seg[tid], mx, inv_t) : 0.f;
        const float before = block_exclusive_scan(mine, L, &total);
        target = u * total;
        if (mine > 0.f && before + mine > target) atomicMin(&L.best, tid);
        __syncthreads();
        s = L.best;
        if (s != 0x7fffffff && tid == s) L.bcast[1] = before;
        __syncthreads();
    }
    int tok = -1;
    if (s != 0x7fffffff) {
        // walk the segment: thread t owns consecutive ids, added up in id order
        const int per = (seg_ids + kSampleThreads - 1) / kSampleThreads;
        const int end = min(V, (s + 1) * seg_ids), j0 = min(end, s * seg_ids + tid * per), j1 = min(end, j0 + per);
        constexpr int kKeep = kSegIds / kSampleThreads;      // weights that are kept (longer segments form them again)
        float x[kKeep], local = 0.f;
        int last = -1;
#pragma unroll
        for (int i = 0; i < kKeep; ++i) x[i] = j0 + i < j1 ? w(j0 + i) : 0.f;
#pragma unroll
        for (int i = 0; i < kKeep; ++i) {
            local += x[i];
            if (x[i] > 0.f) last = j0 + i;
        }
        for (int j = j0 + kKeep; j < j1; ++j) {
            const float y = w(j);
            local += y;
            if (y > 0.f) last = j;
        }
        float seg_total;
        const float at = L.bcast[1] + block_exclusive_scan(local, L, &seg_total);
        if (tid == 0) L.best = 0x7fffffff;
        __syncthreads();
        if (at + local > target || at > target) {
            float c = at;
            int hit = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < kKeep; ++i) {
                c += x[i];
                if (c > target && x[i] > 0.f && hit == 0x7fffffff) hit = j0 + i;
            }
            for (int j = j0 + kKeep; j < j1 && hit == 0x7fffffff; ++j) {
                const float y = w(j);
                c += y;
                if (c > target && y > 0.f) hit = j;
            }
            if (hit != 0x7fffffff) atomicMin(&L.best, hit);
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
    __device__ __forceinline__ float weight(float a, float b) const { return a > b ? expf(a - c) * -expm1f(b - a) : 0.f; }
    __device__ __forceinline__ float operator()(int j) const { return weight(log_p(j), log_q(j)); }
};

// Statistics of the ids [j0, j1) of a row, to every thread
__device__ __forceinline__ SegStat segment_stat(const float *z, int j0, int j1, float inv_t, SampleLds &L) {
    constexpr int kKeep = kSegIds / kSampleThreads;          // values that are kept (longer segments read them again)
    float v[kKeep], m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int j = j0 + (int)threadIdx.x + i * kSampleThreads;
        v[i] = j < j1 ? z[j] : -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < kKeep; ++i) m = fmaxf(m, v[i]);
    for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads) m = fmaxf(m, z[j]);
    m = block_max(m, L);
    float s = 0.f;
    if (m != -INFINITY) {
#pragma unroll
        for (int i = 0; i < kKeep; ++i) s += expf((v[i] - m) * inv_t);
        for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads) s += expf((z[j] - m) * inv_t);
    } else {
        // nothing but -inf, whose weight is 0, and values that are no numbers (fmaxf passes them by): those stay in the sum
#pragma unroll
        for (int i = 0; i < kKeep; ++i)
            if (v[i] != v[i]) s = v[i];
        for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads)
            if (z[j] != z[j]) s = z[j];
    }
    float total;
    (void)block_exclusive_scan(s, L, &total);
    return SegStat{m, total};
}

// Segment blockIdx.x of row blockIdx.y: rows [0, n_first) start at z0, the others at z1.
struct SegArgs { const float *z0, *z1; int n_first, V, n_seg, seg_ids; float inv_t; SegStat *out; };

__global__ void __launch_bounds__(kSampleThreads) k_segment_stats(SegArgs a) {
    __shared__ SampleLds L;
    const int r = blockIdx.y, j0 = blockIdx.x * a.seg_ids;
    const float *z = r < a.n_first ? a.z0 + (size_t)r * a.V : a.z1 + (size_t)(r - a.n_first) * a.V;
    const SegStat st = segment_stat(z, j0, min(a.V, j0 + a.seg_ids), a.inv_t, L);
    if (threadIdx.x == 0) a.out[(size_t)r * a.n_seg + blockIdx.x] = st;
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

// seg: the segments' statistics, or null for a row of one segment, whose statistics are formed here (one kernel less)
__global__ void __launch_bounds__(kSampleThreads) k_sample_row(SampleArgs a, const SegStat *seg, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    __shared__ SegStat only;
    if (!seg) {
        const SegStat st = segment_stat(a.z, 0, a.V, a.inv_t, L);
        if (threadIdx.x == 0) only = st;
        __syncthreads();
        seg = &only;
    }
    const float mx = block_max((int)threadIdx.x < n_seg ? seg[threadIdx.x].mx : -INFINITY, L);
    float w_tok, total;
    const int tok = sample_segments(SoftmaxWeight{a.z, mx, a.inv_t}, seg, mx, a.inv_t, a.V, n_seg, seg_ids, a.u, L, &w_tok, &total);
    if (threadIdx.x == 0) {
        *a.tok_out = tok;
        *a.prob_out = w_tok / total;
    }
}

// The same of a row of one segment, straight from its logits.
__device__ __forceinline__ SegStat row_from_logits(const float *z, int V, float inv_t) {
    const int lane = threadIdx.x & 63;
    float v[kSegIds / 64], m = -INFINITY, s = 0.f;
#pragma unroll
    for (int i = 0; i < kSegIds / 64; ++i) {
        v[i] = lane + 64 * i < V ? z[lane + 64 * i] : -INFINITY;
        m = fmaxf(m, v[i]);
    }
    m = wave_max(m);
    if (m != -INFINITY) {
#pragma unroll
        for (int i = 0; i < kSegIds / 64; ++i) s += expf((v[i] - m) * inv_t);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    return SegStat{m, s};
}

// Eq. 2 over the drafts, computed by every workgroup that needs the outcome (the same sums in the same order).
struct Decision { int n_acc, rejected; SegStat f, q; };      // of row n_acc: statistics of its final and draft logits

// Where the rows' statistics come from.  A kernel is built for one source: in one kernel for all, which also reduced the rows of one
// segment, 5 and 8 rows of 2048 logits took 37.9 us a call and not 36.1.
enum RowSource { ROWS_LOGITS, ROWS_SEGMENT, ROWS_SEGMENTS };     // the logits, one segment per row, several

template <RowSource SRC>
__device__ __forceinline__ Decision decide(const VerifySampledArgs &a, const SegStat *seg, int n_seg, bool write_ratio) {
    __shared__ SegStat row[16];
    __shared__ int s_rejected;                       // the first rejected draft, n_draft if none is
    const int wave = threadIdx.x >> 6, n_draft = a.m - 1;
    const int n_rows = 2 * a.m - 1;
    if (SRC == ROWS_SEGMENT) {
        if ((int)threadIdx.x < n_rows) row[threadIdx.x] = seg[threadIdx.x];
    } else if (SRC == ROWS_SEGMENTS) {
        for (int r = wave; r < n_rows; r += kSampleWaves) {
            const SegStat st = row_from_segments(seg + (size_t)r * n_seg, n_seg, a.inv_t);
            if ((threadIdx.x & 63) == 0) row[r] = st;
        }
    } else if (wave < n_rows) {                      // (at most a row per wavefront)
        const int r = wave;
        const SegStat st = row_from_logits(r < a.m ? a.zf + (size_t)r * a.V : a.zq + (size_t)(r - a.m) * a.V, a.V, a.inv_t);
        if ((threadIdx.x & 63) == 0) row[r] = st;
    }
    // a lane per draft
    const int k = threadIdx.x, t = k < n_draft ? a.draft[k] : 0;
    const float zf = k < n_draft ? a.zf[(size_t)k * a.V + t] : 0.f, zq = k < n_draft ? a.zq[(size_t)k * a.V + t] : 0.f;
    __syncthreads();
    if (wave == 0) {
        float ratio = 0.f;
        bool rejected = false;
        if (k < n_draft) {
            // p*(t) / p_draft(t) through the logarithms, so that two tiny probabilities still have a ratio
            const float lp = (zf - row[k].mx) * a.inv_t - logf(row[k].sum), lq = (zq - row[a.m + k].mx) * a.inv_t - logf(row[a.m + k].sum);
            ratio = expf(lp - lq);
            rejected = !(a.u_accept[k] < fminf(1.0f, ratio));
        }
        const unsigned long long mask = __ballot(rejected);
        const int first = mask ? __ffsll(mask) - 1 : n_draft;
        if (k == 0) s_rejected = first;
        if (write_ratio && a.ratio_out && k < n_draft) a.ratio_out[k] = k <= first ? ratio : 0.f;
    }
    __syncthreads();
    Decision d;
    d.n_acc = s_rejected;
    d.rejected = s_rejected < n_draft;
    d.f = row[d.n_acc];
    d.q = d.rejected ? row[a.m + d.n_acc] : SegStat{0.f, 0.f};
    return d;
}

__device__ __forceinline__ ResidualWeight residual_of(const VerifySampledArgs &a, const Decision &d) {
    return ResidualWeight{a.zf + (size_t)d.n_acc * a.V, a.zq + (size_t)d.n_acc * a.V, d.f.mx, logf(d.f.sum), d.q.mx, logf(d.q.sum), a.inv_t, 0.f};
}

// Statistics of the ids [j0, j1) of the residual: (largest log p* where p* exceeds p_draft, sum of the weights relative to
// it), to every thread.
__device__ __forceinline__ SegStat residual_stat(ResidualWeight w, int j0, int j1, SampleLds &L) {
    constexpr int kKeep = kSegIds / kSampleThreads;          // ids whose log-probabilities are kept (longer segments form them again)
    float la[kKeep], lb[kKeep], c = -INFINITY;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int j = j0 + (int)threadIdx.x + i * kSampleThreads;
        la[i] = j < j1 ? w.log_p(j) : -INFINITY;
        lb[i] = j < j1 ? w.log_q(j) : -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (la[i] > lb[i]) c = fmaxf(c, la[i]);
    for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads) {
        const float a = w.log_p(j);
        if (a > w.log_q(j)) c = fmaxf(c, a);
    }
    w.c = block_max(c, L);
    float s = 0.f;
    if (w.c != -INFINITY) {
#pragma unroll
        for (int i = 0; i < kKeep; ++i) s += w.weight(la[i], lb[i]);
        for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads) s += w(j);
    }
    float total;
    (void)block_exclusive_scan(s, L, &total);
    return SegStat{w.c, total};
}

// The residual's segments, if a draft was rejected.
__global__ void __launch_bounds__(kSampleThreads) k_residual_segments(VerifySampledArgs a, const SegStat *seg, int n_seg, int seg_ids, SegStat *out) {
    __shared__ SampleLds L;
    const Decision d = decide<ROWS_SEGMENTS>(a, seg, n_seg, false);
    if (!d.rejected) return;
    const int j0 = blockIdx.x * seg_ids;
    const SegStat st = residual_stat(residual_of(a, d), j0, min(a.V, j0 + seg_ids), L);
    if (threadIdx.x == 0) out[blockIdx.x] = st;
}

// seg: null for ROWS_LOGITS; res_seg: null but for ROWS_SEGMENTS (a residual of one segment is formed here)
template <RowSource SRC>
__global__ void __launch_bounds__(kSampleThreads) k_verify_sampled(VerifySampledArgs a, const SegStat *seg, const SegStat *res_seg, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    __shared__ SegStat only;
    const Decision d = decide<SRC>(a, seg, n_seg, true);
    const int r = d.n_acc;
    int tok = -1;
    float w_tok, total;
    if (d.rejected) {
        ResidualWeight w = residual_of(a, d);
        if (SRC != ROWS_SEGMENTS) {
            const SegStat st = residual_stat(w, 0, a.V, L);
            if (threadIdx.x == 0) only = st;
            __syncthreads();
            res_seg = &only;
        }
        w.c = block_max((int)threadIdx.x < n_seg ? res_seg[threadIdx.x].mx : -INFINITY, L);
        if (w.c != -INFINITY) tok = sample_segments(w, res_seg, w.c, 1.0f, a.V, n_seg, seg_ids, a.u_resample[r], L, &w_tok, &total);
        __syncthreads();
    }
    const SegStat *row_seg = &only;
    if (SRC == ROWS_SEGMENTS) {
        row_seg = seg + (size_t)r * n_seg;
    } else {
        __syncthreads();
        if (threadIdx.x == 0) only = d.f;
        __syncthreads();
    }
    if (tok < 0)       // nothing rejected (or a residual that is identically zero): draw from the row's final distribution
        tok = sample_segments(SoftmaxWeight{a.zf + (size_t)r * a.V, d.f.mx, a.inv_t}, row_seg, d.f.mx, a.inv_t, a.V, n_seg, seg_ids,
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
    SegStat *seg = n_seg > 1 ? (SegStat *)a.scratch : nullptr;
    if (seg) hipLaunchKernelGGL(k_segment_stats, dim3(n_seg, 1), dim3(kSampleThreads), 0, (hipStream_t)stream,
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
    SegStat *seg = nullptr, *res_seg = nullptr;
    const dim3 wg(kSampleThreads);
    int rc;
    // rows of one segment: up to as many as a workgroup has wavefronts are cheaper to reduce in the last kernel than in one of
    // their own (2048 logits, 3 rows: 33.6 against 35.4 us a call; more take a kernel of their own, one kernel for 15 rows took
    // 39.5 against 38.2), and the residual always is
    if (n_seg > 1 || 2 * a.m - 1 > kSampleWaves) {
        seg = (SegStat *)a.scratch;
        hipLaunchKernelGGL(k_segment_stats, dim3(n_seg, 2 * a.m - 1), wg, 0, (hipStream_t)stream, SegArgs{a.zf, a.zq, a.m, a.V, n_seg, seg_ids, a.inv_t, seg});
        if ((rc = (int)hipGetLastError())) return rc;
    }
    if (n_seg > 1 && a.m > 1) {
        res_seg = seg + (size_t)(2 * a.m - 1) * n_seg;
        hipLaunchKernelGGL(k_residual_segments, dim3(n_seg), wg, 0, (hipStream_t)stream, a, seg, n_seg, seg_ids, res_seg);
        if ((rc = (int)hipGetLastError())) return rc;
    }
    if (n_seg > 1) hipLaunchKernelGGL(k_verify_sampled<ROWS_SEGMENTS>, dim3(1), wg, 0, (hipStream_t)stream, a, seg, res_seg, n_seg, seg_ids);
    else if (seg) hipLaunchKernelGGL(k_verify_sampled<ROWS_SEGMENT>, dim3(1), wg, 0, (hipStream_t)stream, a, seg, res_seg, n_seg, seg_ids);
    else hipLaunchKernelGGL(k_verify_sampled<ROWS_LOGITS>, dim3(1), wg, 0, (hipStream_t)stream, a, seg, res_seg, n_seg, seg_ids);
    return (int)hipGetLastError();
}

}  // namespace ad
