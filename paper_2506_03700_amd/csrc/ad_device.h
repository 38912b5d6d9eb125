// Device-side helpers shared by the library's kernels: vector types, bf16 conversion, and the index
// function of the packed activation layout (see ad_internal.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ad {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;   // also carries 8 fp16 values (see mma16)
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// ---------------------------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round-to-nearest-even fp32 -> bf16 bits (finite inputs)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float f16_bits_to_f32(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }

// Kernel arguments are fetched with scalar loads that the compiler places where each field is first used; every
// 64-byte line of the argument block that is touched for the first time costs a trip to memory, and those trips
// come one after the other on the path to the kernel's first useful load.  Reading one word of every line of the
// block at the kernel's entry (and waiting for them together) overlaps them all: later argument loads hit in the
// scalar cache.  BYTES: the size of the kernel's explicit arguments; nothing beyond them is read.
// threadIdx.x as a value the compiler computes afresh at every call.  The phases of a kernel that loops over layers
// derive their lane-dependent addresses from it: derived from threadIdx.x itself they would all count as loop
// invariants, be computed ahead of the loop and be kept in registers (spilled, there are hundreds) through every phase.
__device__ __forceinline__ int thread_index() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Declares the registers of an array to hold nothing that is still needed (no instruction is emitted).  Inside a
// loop, an array that is only filled under a condition would otherwise carry its contents of the previous turn
// all the way round the loop.
template <class T, int A>
__device__ __forceinline__ void forget(T (&r)[A]) {
#pragma unroll
    for (int i = 0; i < A; ++i) asm volatile("" : "=v"(r[i]));
}
template <class T, int A, int B>
__device__ __forceinline__ void forget(T (&r)[A][B]) {
#pragma unroll
    for (int i = 0; i < A; ++i) forget(r[i]);
}

template <int BYTES>
__device__ __forceinline__ void warm_kernel_args() {
    typedef const __attribute__((address_space(4))) uint32_t *kptr;
    kptr p = (kptr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (BYTES + 63) / 64;
    uint32_t v[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) v[i] = p[i * 16 < BYTES / 4 ? i * 16 : BYTES / 4 - 1];
#pragma unroll
    for (int i = 0; i < LINES; ++i) asm volatile("" ::"s"(v[i]));
}

// The same without the wait: `use` goes where the words are to have arrived.  For kernels whose first loads need nothing but leading scalar
// parameters, of which the compiler has the first 14 words put into registers before a wavefront starts (-amdgpu-kernarg-preload-count):
// the trip to memory for the others then passes beside those loads.  Layer step of the 8B shape, 1 / 5 rows 87.8 -> 86.4, 93.8 -> 92.0 us, four
// fp16 layers 352 -> 346, the GPU's part of a tiny fp32 token 73.9 -> 67.4 (projections and the fold of the attention splits; the attention
// kernels themselves gained nothing).
template <int BYTES>
struct KernelArgLines {
    static constexpr int LINES = (BYTES + 63) / 64;
    uint32_t v[LINES];
    __device__ __forceinline__ KernelArgLines() {
        typedef const __attribute__((address_space(4))) uint32_t *kptr;
        kptr p = (kptr)__builtin_amdgcn_kernarg_segment_ptr();
#pragma unroll
        for (int i = 0; i < LINES; ++i) v[i] = p[i * 16 < BYTES / 4 ? i * 16 : BYTES / 4 - 1];
    }
    __device__ __forceinline__ void use() const {
#pragma unroll
        for (int i = 0; i < LINES; ++i) asm volatile("" ::"s"(v[i]));
    }
};

// Element kinds of stored tensors (weights, norm vectors, embedding table, KV cache).  16-bit activations use
// the same type as the weights they meet in an MFMA: bf16 for fp32 and bf16 models, fp16 for fp16 models.
enum ElemKind : int { ELEM_F32 = 0, ELEM_BF16 = 1, ELEM_F16 = 2 };

typedef __attribute__((__vector_size__(4 * sizeof(uint16_t)))) uint16_t u16x4;
typedef __attribute__((__vector_size__(8 * sizeof(uint16_t)))) uint16_t u16x8;

// fp32 -> 16 bits (F16: half precision, else bf16); the conversion instructions round to nearest even
template <bool F16>
__device__ __forceinline__ uint16_t to16(float v) {
    if constexpr (F16) return __builtin_bit_cast(uint16_t, (_Float16)v);
    else return __builtin_bit_cast(uint16_t, (__bf16)v);
}
template <bool F16>
__device__ __forceinline__ float from16(uint16_t b) { return F16 ? f16_bits_to_f32(b) : bf16_bits_to_f32(b); }
// v = hi + lo.  For fp16 v is rounded to fp32 before it is split: as a product it could otherwise be fused into one of the
// two uses of hi (a multiplication that rounds to fp16 at once) and not into the other, and at a tie the two would differ.
template <bool F16>
__device__ __forceinline__ void split16(float v, uint16_t &hi, uint16_t &lo) {
    if constexpr (F16) asm("" : "+v"(v));
    hi = to16<F16>(v);
    lo = to16<F16>(v - from16<F16>(hi));
}

// The same for bf16 in the fused layer step, with the rounding in integer arithmetic (same bits for
// finite values): with the conversion instruction the fused step is 1 % slower at one row (8B shape, context 4096: 98.7 -> 99.7 us
// a layer; 8 rows 117.1 -> 116.6).
__device__ __forceinline__ void split_hi_lo(float x, uint16_t &hi, uint16_t &lo) {
    hi = f32_to_bf16_bits(x);
    lo = f32_to_bf16_bits(x - bf16_bits_to_f32(hi));
}

// The value that scores are taken relative to in a softmax: their maximum m, or 0 where every score so far is minus
// infinity (a key whose entry in the cache overflowed): exp(-inf - 0) gives such keys the weight 0, exp(-inf - m) is not a number.
__device__ __forceinline__ float softmax_ref(float m) { return m == -INFINITY ? 0.f : m; }

// ---- sums, maxima and scans over a wavefront, in register moves between lanes (no trip through LDS) ----
// v of the lane that DPP control CTRL names; `none` where there is no such lane
template <int CTRL>
__device__ __forceinline__ float dpp(float v, float none = 0.f) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float read_lane(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
// sum over the 8 lanes of an aligned group of 8
__device__ __forceinline__ float sum8(float v) {
    v += dpp<0xB1>(v);           // quad_perm [1, 0, 3, 2]
    v += dpp<0x4E>(v);           // quad_perm [2, 3, 0, 1]
    return v + dpp<0x141>(v);    // row_half_mirror: the other four
}
// sum over the wavefront
__device__ __forceinline__ float sum64(float v) {
    v = sum8(v);
    v += dpp<0x140>(v);          // row_mirror: the other eight of 16
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}
// largest value of the wavefront (values that are no numbers are passed by)
__device__ __forceinline__ float max64(float v) {
    v = fmaxf(v, dpp<0xB1>(v));
    v = fmaxf(v, dpp<0x4E>(v));
    v = fmaxf(v, dpp<0x141>(v));
    v = fmaxf(v, dpp<0x140>(v));
    return fmaxf(fmaxf(read_lane(v, 0), read_lane(v, 16)), fmaxf(read_lane(v, 32), read_lane(v, 48)));
}
// largest value, and sum, over the four lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ void across_rows(float v, float &a, float &b, float &c, float &e) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const auto q = __builtin_amdgcn_permlane16_swap(p[0], p[0], false, false), r = __builtin_amdgcn_permlane16_swap(p[1], p[1], false, false);
    a = __uint_as_float(q[0]);
    b = __uint_as_float(q[1]);
    c = __uint_as_float(r[0]);
    e = __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_rows(float v) {
    float a, b, c, e;
    across_rows(v, a, b, c, e);
    return fmaxf(fmaxf(a, b), fmaxf(c, e));
}
__device__ __forceinline__ float sum_rows(float v) {
    float a, b, c, e;
    across_rows(v, a, b, c, e);
    return (a + b) + (c + e);
}
// smallest value of the wavefront
__device__ __forceinline__ int min64(int v) {
    auto m = [](int x, int y) { return x < y ? x : y; };
    v = m(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false));
    v = m(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false));
    v = m(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));
    v = m(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false));
    return m(m(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), m(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
// sum over the lanes before this one; *total: over all
__device__ __forceinline__ float scan64(float v, int lane, float *total) {
    float in = v;                // inclusive within a row of 16 lanes
    in += dpp<0x111>(in);        // row_shr 1, 2, 4, 8
    in += dpp<0x112>(in);
    in += dpp<0x114>(in);
    in += dpp<0x118>(in);
    const float r0 = read_lane(in, 15), r1 = r0 + read_lane(in, 31), r2 = r1 + read_lane(in, 47);
    *total = r2 + read_lane(in, 63);
    const float ex = dpp<0x111>(in);
    const int row = lane >> 4;
    return ex + (row == 0 ? 0.f : row == 1 ? r0 : row == 2 ? r1 : r2);
}

// merges (max, sum of exp relative to it, argmax); the lower index wins among equal values
__device__ __forceinline__ void max_merge(float &M, float &S, int &I, float m2, float s2, int i2) {
    if (m2 > M || (m2 == M && i2 < I)) I = i2;
    const float nm = fmaxf(M, m2), ref = softmax_ref(nm);
    S = S * __expf(M - ref) + s2 * __expf(m2 - ref);
    M = nm;
}

// ---- what the workgroups of a launch leave for the last of them ----
// Relaxed agent-scope accesses: stores go through to memory and loads do not use a stale copy in another XCD's L2.
__device__ __forceinline__ void publish(float *p, f32x2 v) {
    __hip_atomic_store((uint64_t *)p, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2 published(const float *p) {
    return __builtin_bit_cast(f32x2, __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// Called by every thread of each of n workgroups (n the same for all launches on this counter) when its wavefront 0 has published what
// the workgroup leaves: true in the workgroup that is the last to call, where all of it can be read.  Nobody waits for another workgroup.
// The counter counts modulo n, so that it is back at 0 when the launch ends (and also after launches that ran at the same time, whose outcomes are
// then anybody's).  In place of a second kernel it saves 1.5 to 2 us behind 63 workgroups (a draw from 128256 logits, a sampled verification), and
// nothing behind the 256 of a vocabulary pass, whose arrivals take as long as the launch did.
__device__ __forceinline__ bool last_to_arrive(unsigned *counter, unsigned n, int *shared) {
    if (threadIdx.x < 64) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // what this wavefront has published is in memory
        if (threadIdx.x == 0) *shared = atomicInc(counter, n - 1) == n - 1;
    }
    __syncthreads();
    return *shared;
}

// A result for the host: written through to (pinned, uncached) memory.  done: the word that the host watches, behind the results that this wavefront
// has reported (those of others have to be in memory before: reported, and then a barrier).  A release store would write the L2's dirty
// lines back first, which nothing here needs.
__device__ __forceinline__ void report(int32_t *p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ __forceinline__ void report(float *p, float v) { report((int32_t *)p, __float_as_int(v)); }
__device__ __forceinline__ void reported() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void report_done(int32_t *flag, int32_t seq) {
    if (!flag) return;
    reported();
    report(flag, seq);
}

// D += A (16 rows x 32) * B (32 x 16 columns), 16-bit operands of the model's type, fp32 accumulation
template <bool F16>
__device__ __forceinline__ f32x4 mma16(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float load_w(const void *p, int elem, size_t i) {
    if (elem == ELEM_F32) return ((const float *)p)[i];
    const uint16_t b = ((const uint16_t *)p)[i];
    return elem == ELEM_BF16 ? bf16_bits_to_f32(b) : f16_bits_to_f32(b);
}

// eight consecutive weights starting at element k (k a multiple of 8); a null vector means all ones
__device__ __forceinline__ void load_w8(const void *p, int elem, size_t k, float (&w)[8]) {
    if (!p) {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = 1.0f;
    } else if (elem == ELEM_BF16) {
        const u32x4 v = *(const u32x4 *)((const uint16_t *)p + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[2 * e] = __uint_as_float(v[e] << 16);
            w[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
        }
    } else if (elem == ELEM_F16) {
        const u32x4 v = *(const u32x4 *)((const uint16_t *)p + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[2 * e] = f16_bits_to_f32((uint16_t)(v[e] & 0xffffu));
            w[2 * e + 1] = f16_bits_to_f32((uint16_t)(v[e] >> 16));
        }
    } else {
        const f32x4 v0 = *(const f32x4 *)((const float *)p + k), v1 = *(const f32x4 *)((const float *)p + k + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[e] = v0[e];
            w[4 + e] = v1[e];
        }
    }
}

// v + (v of the lane 8 places away within its group of 16 lanes): the hi and lo columns of an MFMA result.
// A DPP row rotation by 8, so it costs one VALU instruction and no LDS traffic.
__device__ __forceinline__ float add_lane_xor8(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128 /* row_ror:8 */, 0xf, 0xf, false);
    return v + __int_as_float(o);
}

// x / d for small non-negative x and d, with the multiplier the host derived from d (div_multiplier in ad_internal.h)
// (a multiplier of 0 stands for d == 1)
__device__ __forceinline__ int div_small(int x, unsigned mul) { return mul ? (int)__umulhi((unsigned)x, mul) : x; }

// index (in bf16 elements) of input k of column col (token col & 7, hi/lo part col >> 3) in a packed activation
// block of KT k-steps (see ad_internal.h)
__device__ __forceinline__ size_t act_index(int k, int col, int KT) {
    return ((((size_t)(col & 7) * KT + (k >> 5)) * 2 + (col >> 3)) * 4 + ((k & 31) >> 3)) * 8 + (k & 7);
}

// v as input k of token t in a packed activation block of KT k-steps
template <bool F16>
__device__ __forceinline__ void store_act(void *B, int KT, int k, int t, float v) {
    uint16_t hi, lo;
    split16<F16>(v, hi, lo);
    ((uint16_t *)B)[act_index(k, t, KT)] = hi;
    ((uint16_t *)B)[act_index(k, 8 + t, KT)] = lo;
}

// index (in 16-byte units) of the MFMA B operand register of lane `lane` for k-step ks of such a block
__device__ __forceinline__ size_t act_operand_index(int ks, int lane, int KT) {
    const int n = lane & 15;
    return (((size_t)(n & 7) * KT + ks) * 2 + (n >> 3)) * 4 + (lane >> 4);
}

}  // namespace ad
