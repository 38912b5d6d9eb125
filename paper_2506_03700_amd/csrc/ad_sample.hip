// Sampled decoding (Sec. 2.2 of arxiv 2506.03700): the token of Eq. 1 drawn from softmax(z / T), and the
// verification of Eq. 2 in its general form -- a drafted token t survives with probability
// min(1, p*(t) / p_draft(t)); the first rejected draft is replaced by a draw from
// Normalize(max(0, p* - p_draft)); if none is rejected the next token is drawn from the newest row's p*.
//
// Every draw is a uniform number u in [0, 1) handed in by the caller and turned into a token by inversion of
// the cumulative distribution in token-id order: the first id whose cumulative weight exceeds u * (total
// weight).  A row is cut into segments of consecutive ids, one workgroup each, which leaves its segment's maximum
// and sum of weights; the last workgroup to arrive finds the segment that holds the target from those (in every wavefront at once)
// and walks that segment alone.  What bounds these calls is not the row (0.5 MB) but the chain of dependent loads, reductions and kernel
// boundaries: with one workgroup that passed over the whole row three times a draw from 128256 logits took 97 us on the
// GPU, with segments and every reduction and scan through LDS 12.5, now that they move between registers and the wavefronts repeat
// what is small instead of waiting for one of them 6.4 (a call 31.8 -> 26.2; verification of 6 rows 21.3 -> 15.1, a call 46.9 ->
// 37.4); the last workgroup in place of a kernel behind it: a call 16.6 -> 14.8 us, of verification 27.5 -> 25.8; the sums are added up in a fixed order (no float atomics), so everything is deterministic.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_launch.h"

namespace ad {

namespace {

constexpr int kSampleThreads = 512;              // against 256: 4 rows of 128256 logits 35.4, 37.6 us a call, 1 and 8 rows alike
constexpr int kSampleWaves = kSampleThreads / 64;
constexpr int kSegIds = 2048;                    // ids per segment, until there are as many segments as a workgroup has threads

struct SampleLds {
    float wave_val[2][kSampleWaves];
    int wave_id[2][kSampleWaves];
    int last_pos;
    int last_wg;
};

// (largest value, sum of the weights relative to it) of a segment
struct SegStat { float mx, sum; };

// max over the workgroup, returned to every thread (slot: which of the two exchanges in LDS)
__device__ __forceinline__ float block_max(float v, SampleLds &L, int slot) {
    v = max64(v);
    if ((threadIdx.x & 63) == 0) L.wave_val[slot][threadIdx.x >> 6] = v;
    __syncthreads();
    float r = L.wave_val[slot][0];
#pragma unroll
    for (int w = 1; w < kSampleWaves; ++w) r = fmaxf(r, L.wave_val[slot][w]);
    return r;
}

__device__ __forceinline__ float block_sum(float v, SampleLds &L, int slot) {
    v = sum64(v);
    if ((threadIdx.x & 63) == 0) L.wave_val[slot][threadIdx.x >> 6] = v;
    __syncthreads();
    float r = L.wave_val[slot][0];
#pragma unroll
    for (int w = 1; w < kSampleWaves; ++w) r += L.wave_val[slot][w];
    return r;
}

// a segment's sum relative to the row's largest value (a segment without weight has none, whatever its maximum)
__device__ __forceinline__ float rescaled(SegStat s, float mx, float inv_t) {
    return (s.sum == 0.f) ? 0.f : s.sum * expf((s.mx - mx) * inv_t);
}

constexpr int kLaneSegs = kSampleThreads / 64;           // most segments per lane of a wavefront

// A row's segments in the registers of a wavefront (every wavefront of the workgroup does the same, which saves the barriers):
// lane l holds segments l * per .. + per - 1.
struct RowSegs {
    SegStat v[kLaneSegs];
    int per, lane;
    // PUBLISHED: by other workgroups of this launch
    template <bool PUBLISHED = false>
    __device__ __forceinline__ void load(const SegStat *seg, int n_seg) {
        lane = threadIdx.x & 63;
        per = (n_seg + 63) >> 6;
#pragma unroll
        for (int i = 0; i < kLaneSegs; ++i) {
            v[i] = SegStat{-INFINITY, 0.f};
            if (i < per && lane * per + i < n_seg) {
                if constexpr (PUBLISHED) {
                    const f32x2 p = published((const float *)(seg + lane * per + i));
                    v[i] = SegStat{p[0], p[1]};
                } else {
                    v[i] = seg[lane * per + i];
                }
            }
        }
    }
    __device__ __forceinline__ void one(SegStat s) {     // a row of one segment
        lane = threadIdx.x & 63;
        per = 1;
        v[0] = lane == 0 ? s : SegStat{-INFINITY, 0.f};
    }
    __device__ __forceinline__ float max() const {
        float m = v[0].mx;
#pragma unroll
        for (int i = 1; i < kLaneSegs; ++i)
            if (i < per) m = fmaxf(m, v[i].mx);
        return max64(m);
    }
    // turns the sums into weights relative to mx; returns this lane's
    __device__ __forceinline__ float rescale(float mx, float inv_t) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < kLaneSegs; ++i)
            if (i < per) {
                v[i].sum = rescaled(v[i], mx, inv_t);
                s += v[i].sum;
            }
        return s;
    }
};

// What a draw gives every thread: the token (-1: no id of positive weight), the total weight; `owner` is set in the one thread
// that is to report it, with the token's weight w.
struct Draw { int tok; float total, w; bool owner; };

// Inversion draw over the weights w(j) >= 0 of a row whose segments are in `segs`, rescaled (segment's weights are relative to its
// own maximum); `mine`: this lane's share of the total.  The draw is a chain: one wavefront-wide scan finds the segment, its ids
// are loaded, one scan over the workgroup finds the id (two barriers).
template <class W>
__device__ __forceinline__ Draw draw_from(W w, const RowSegs &segs, float mine, int V, int seg_ids, float u, SampleLds &L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float total;
    const float before = scan64(mine, lane, &total), target = u * total;
    Draw d{-1, total, 0.f, false};
    const unsigned long long hits = __ballot(mine > 0.f && before + mine > target);
    if (hits) {
        // the first lane that reaches the target, and in it the first segment that does (the two sums may round differently:
        // then its last segment with weight)
        int s = 0;
        float at_s = before, c = before;
        bool found = false;
#pragma unroll
        for (int i = 0; i < kLaneSegs; ++i)
            if (i < segs.per) {
                if (!found && segs.v[i].sum > 0.f) {
                    s = lane * segs.per + i;
                    at_s = c;
                    found = c + segs.v[i].sum > target;
                }
                c += segs.v[i].sum;
            }
        const int l0 = __ffsll(hits) - 1;
        s = __builtin_amdgcn_readlane(s, l0);
        at_s = read_lane(at_s, l0);
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
        float wave_total;
        float at = scan64(local, lane, &wave_total);
        const unsigned long long live = __ballot(last >= 0);
        if (lane == 0) L.wave_val[0][wave] = wave_total;
        if (live && lane == 63 - __clzll(live)) L.wave_id[0][wave] = last;
        if (!live && lane == 0) L.wave_id[0][wave] = -1;
        __syncthreads();
        float ahead = 0.f;
        int seg_last = -1;
#pragma unroll
        for (int k = 0; k < kSampleWaves; ++k) {
            ahead += k < wave ? L.wave_val[0][k] : 0.f;
            if (L.wave_id[0][k] >= 0) seg_last = L.wave_id[0][k];
        }
        at += at_s + ahead;
        int hit = 0x7fffffff;
        float w_hit = 0.f;
        if (at + local > target || at > target) {
            float c2 = at;
#pragma unroll
            for (int i = 0; i < kKeep; ++i) {
                c2 += x[i];
                if (c2 > target && x[i] > 0.f && hit == 0x7fffffff) {
                    hit = j0 + i;
                    w_hit = x[i];
                }
            }
            for (int j = j0 + kKeep; j < j1 && hit == 0x7fffffff; ++j) {
                const float y = w(j);
                c2 += y;
                if (c2 > target && y > 0.f) {
                    hit = j;
                    w_hit = y;
                }
            }
        }
        // the wavefront's lowest id (its first lane with one), then the lowest of the wavefronts'
        const unsigned long long got = __ballot(hit != 0x7fffffff);
        const int wave_hit = got ? __builtin_amdgcn_readlane(hit, __ffsll(got) - 1) : 0x7fffffff;
        if (lane == 0) L.wave_id[1][wave] = wave_hit;
        __syncthreads();
        int tok = 0x7fffffff;
#pragma unroll
        for (int k = 0; k < kSampleWaves; ++k) tok = min(tok, L.wave_id[1][k]);
        if (tok != 0x7fffffff) {
            d.tok = tok;
            d.w = w_hit;
            d.owner = hit == tok;
        } else if (seg_last >= 0) {
            // the two ways of adding the segment up may round differently: then its last id of positive weight
            d.tok = seg_last;
            d.owner = tid == 0;
            if (d.owner) d.w = w(seg_last);
        }
    }
    if (d.tok < 0) {
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
        d.tok = L.last_pos;
        d.owner = tid == 0;
        d.w = d.owner && d.tok >= 0 ? w(d.tok) : 0.f;
    }
    return d;
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
    m = block_max(m, L, 0);
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
    return SegStat{m, block_sum(s, L, 1)};
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

// (max z, sum exp((z - max) * inv_t)) of a row from its segments, by one wavefront
__device__ __forceinline__ SegStat row_from_segments(RowSegs &segs, float inv_t) {
    const float m = segs.max();
    return SegStat{m, sum64(segs.rescale(m, inv_t))};
}

// A workgroup per segment; the last one to arrive draws.
__global__ void __launch_bounds__(kSampleThreads) k_sample_row(SampleArgs a, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    const int j0 = blockIdx.x * seg_ids;
    const SegStat st = segment_stat(a.z, j0, min(a.V, j0 + seg_ids), a.inv_t, L);
    RowSegs segs;
    if (n_seg == 1) {
        segs.one(st);
        __syncthreads();
    } else {
        SegStat *seg = (SegStat *)a.scratch;
        if (threadIdx.x == 0) publish((float *)(seg + blockIdx.x), (f32x2){st.mx, st.sum});
        if (!last_to_arrive(a.arrivals, n_seg, &L.last_wg)) return;
        segs.load<true>(seg, n_seg);
    }
    const float mx = segs.max(), mine = segs.rescale(mx, a.inv_t);
    const Draw d = draw_from(SoftmaxWeight{a.z, mx, a.inv_t}, segs, mine, a.V, seg_ids, a.u, L);
    if (d.owner) {
        report(a.tok_out, d.tok);
        if (a.prob_out) report(a.prob_out, d.w / d.total);
        if (a.n_accept_out) report(a.n_accept_out, 0);
        report_done(a.done_flag, a.done_seq);
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
    m = max64(m);
    if (m != -INFINITY) {
#pragma unroll
        for (int i = 0; i < kSegIds / 64; ++i) s += expf((v[i] - m) * inv_t);
    }
    return SegStat{m, sum64(s)};
}

// Eq. 2 over the drafts, computed by every workgroup that needs the outcome (the same sums in the same order).
struct Decision { int n_acc, rejected; SegStat f, q; };      // of row n_acc: statistics of its final and draft logits

// Where the rows' statistics come from.  A kernel is built for one source: one kernel for all, which also reduced the rows of one
// segment, took 37.9 us a call for 5 and 8 rows of 2048 logits when three kernels took 36.1 (31.7 now).
enum RowSource { ROWS_LOGITS, ROWS_SEGMENT, ROWS_SEGMENTS };     // the logits, one segment per row, several

// *ratio: of draft `lane` (0 if it was not checked), the same in every wavefront
template <RowSource SRC>
__device__ __forceinline__ Decision decide(const VerifySampledArgs &a, const SegStat *seg, int n_seg, float *ratio_out) {
    __shared__ SegStat row[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_draft = a.m - 1, n_rows = 2 * a.m - 1;
    // a lane per draft, in every wavefront
    const int k = lane, t = k < n_draft ? a.draft[k] : 0;
    const float zf = k < n_draft ? a.zf[(size_t)k * a.V + t] : 0.f, zq = k < n_draft ? a.zq[(size_t)k * a.V + t] : 0.f;
    if (SRC == ROWS_SEGMENT) {
        if ((int)threadIdx.x < n_rows) row[threadIdx.x] = seg[threadIdx.x];
    } else if (SRC == ROWS_SEGMENTS) {
        RowSegs s0, s1;                              // at most two rows per wavefront
        const int r1 = wave + kSampleWaves;
        if (wave < n_rows) s0.load(seg + (size_t)wave * n_seg, n_seg);
        if (r1 < n_rows) s1.load(seg + (size_t)r1 * n_seg, n_seg);
        if (wave < n_rows) {
            const SegStat st = row_from_segments(s0, a.inv_t);
            if (lane == 0) row[wave] = st;
        }
        if (r1 < n_rows) {
            const SegStat st = row_from_segments(s1, a.inv_t);
            if (lane == 0) row[r1] = st;
        }
    } else if (wave < n_rows) {                      // (at most a row per wavefront)
        const int r = wave;
        const SegStat st = row_from_logits(r < a.m ? a.zf + (size_t)r * a.V : a.zq + (size_t)(r - a.m) * a.V, a.V, a.inv_t);
        if (lane == 0) row[r] = st;
    }
    __syncthreads();
    float ratio = 0.f;
    bool rejected = false;
    if (k < n_draft) {
        // p*(t) / p_draft(t) through the logarithms, so that two tiny probabilities still have a ratio
        const float lp = (zf - row[k].mx) * a.inv_t - logf(row[k].sum), lq = (zq - row[a.m + k].mx) * a.inv_t - logf(row[a.m + k].sum);
        ratio = expf(lp - lq);
        rejected = !(a.u_accept[k] < fminf(1.0f, ratio));
    }
    const unsigned long long mask = __ballot(rejected);
    Decision d;
    d.n_acc = mask ? __ffsll(mask) - 1 : n_draft;    // the first rejected draft, n_draft if none is
    d.rejected = d.n_acc < n_draft;
    *ratio_out = k <= d.n_acc ? ratio : 0.f;
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
    w.c = block_max(c, L, 0);
    float s = 0.f;
    if (w.c != -INFINITY) {
#pragma unroll
        for (int i = 0; i < kKeep; ++i) s += w.weight(la[i], lb[i]);
        for (int j = j0 + (int)threadIdx.x + kKeep * kSampleThreads; j < j1; j += kSampleThreads) s += w(j);
    }
    return SegStat{w.c, block_sum(s, L, 1)};
}

// Everything from the rows' statistics on.  ROWS_SEGMENTS: every workgroup takes the decision and, if a draft was rejected, reduces its segment of
// the residual; the last one to arrive draws.  Otherwise one workgroup does it all (seg: null for ROWS_LOGITS).
template <RowSource SRC>
__global__ void __launch_bounds__(kSampleThreads) k_verify_sampled(VerifySampledArgs a, const SegStat *seg, SegStat *res_seg, int n_seg, int seg_ids) {
    __shared__ SampleLds L;
    RowSegs segs;
    float ratio;
    const Decision d = decide<SRC>(a, seg, n_seg, &ratio);
    const int r = d.n_acc;
    Draw dr{-1, 0.f, 0.f, false};
    if (d.rejected) {
        ResidualWeight w = residual_of(a, d);
        if (SRC == ROWS_SEGMENTS) {
            const int j0 = blockIdx.x * seg_ids;
            const SegStat st = residual_stat(w, j0, min(a.V, j0 + seg_ids), L);
            if (threadIdx.x == 0) publish((float *)(res_seg + blockIdx.x), (f32x2){st.mx, st.sum});
            if (!last_to_arrive(a.arrivals, n_seg, &L.last_wg)) return;
            segs.load<true>(res_seg, n_seg);
        } else {
            segs.one(residual_stat(w, 0, a.V, L));
            __syncthreads();
        }
        w.c = segs.max();
        const float mine = segs.rescale(w.c, 1.0f);
        if (w.c != -INFINITY) dr = draw_from(w, segs, mine, a.V, seg_ids, a.u_resample[r], L);
    } else if (SRC == ROWS_SEGMENTS) {
        // here too the last one goes on: once the done word is out, no workgroup that started late still reads rows or statistics that the caller
        // may then be writing on another stream
        __syncthreads();
        if (!last_to_arrive(a.arrivals, n_seg, &L.last_wg)) return;
    }
    if (dr.tok < 0) {  // nothing rejected (or a residual that is identically zero): draw from the row's final distribution
        if (SRC == ROWS_SEGMENTS) segs.load(seg + (size_t)r * n_seg, n_seg);
        else segs.one(d.f);
        __syncthreads();
        const float mine = segs.rescale(d.f.mx, a.inv_t);
        dr = draw_from(SoftmaxWeight{a.zf + (size_t)r * a.V, d.f.mx, a.inv_t}, segs, mine, a.V, seg_ids, d.rejected ? a.u_resample[r] : a.u_final, L);
    }
    // the wavefront that has the token reports everything: its store of the done word is ordered behind its own
    if (a.ratio_out && __any(dr.owner) && (int)(threadIdx.x & 63) < a.m - 1) report(a.ratio_out + (threadIdx.x & 63), ratio);
    if (dr.owner) {
        report(a.n_accept_out, r);
        report(a.next_out, dr.tok);
        report_done(a.done_flag, a.done_seq);
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

int launch_sample_row(const SampleArgs &a, const LaunchCtx &c) {
    if (a.V < 1 || !(a.inv_t > 0.f)) return (int)hipErrorInvalidValue;
    int n_seg, seg_ids;
    segments(a.V, &n_seg, &seg_ids);
    return launch<k_sample_row>(c, dim3(n_seg), dim3(kSampleThreads), 0, a, n_seg, seg_ids);
}

int launch_verify_sampled(const VerifySampledArgs &a, const LaunchCtx &c) {
    if (a.V < 1 || a.m < 1 || a.m > 8 || !(a.inv_t > 0.f)) return (int)hipErrorInvalidValue;
    if (a.m == 1) {                                  // no drafts: a draw from the row
        SampleArgs s;
        s.z = a.zf; s.V = a.V; s.inv_t = a.inv_t; s.u = a.u_final; s.tok_out = a.next_out; s.prob_out = nullptr; s.n_accept_out = a.n_accept_out;
        s.scratch = a.scratch; s.arrivals = a.arrivals; s.done_flag = a.done_flag; s.done_seq = a.done_seq;
        return launch_sample_row(s, c);
    }
    for (int k = 0; k + 1 < a.m; ++k)
        if (a.draft[k] < 0 || a.draft[k] >= a.V) return (int)hipErrorInvalidValue;
    int n_seg, seg_ids;
    segments(a.V, &n_seg, &seg_ids);
    SegStat *seg = nullptr;
    const dim3 wg(kSampleThreads);
    // rows of one segment: up to as many as a workgroup has wavefronts are cheaper to reduce in the last kernel than in one of
    // their own (2048 logits, 3 rows: 28.5 against 29.3 us a call, 4 rows 31.2 / 31.9; more take a kernel of their own), and the
    // residual always is
    if (n_seg > 1 || 2 * a.m - 1 > kSampleWaves) {
        seg = (SegStat *)a.scratch;
        const int rc = launch<k_segment_stats>(c, dim3(n_seg, 2 * a.m - 1), wg, 0, SegArgs{a.zf, a.zq, a.m, a.V, n_seg, seg_ids, a.inv_t, seg});
        if (rc) return rc;
    }
    SegStat *res_seg = n_seg > 1 ? seg + (size_t)(2 * a.m - 1) * n_seg : nullptr;
    if (n_seg > 1) return launch<k_verify_sampled<ROWS_SEGMENTS>>(c, dim3(n_seg), wg, 0, a, (const SegStat *)seg, res_seg, n_seg, seg_ids);
    if (seg) return launch<k_verify_sampled<ROWS_SEGMENT>>(c, dim3(1), wg, 0, a, (const SegStat *)seg, res_seg, n_seg, seg_ids);
    return launch<k_verify_sampled<ROWS_LOGITS>>(c, dim3(1), wg, 0, a, (const SegStat *)seg, res_seg, n_seg, seg_ids);
}

}  // namespace ad
