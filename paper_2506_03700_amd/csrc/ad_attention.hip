// Attention phase of the layer step: rotary embedding of q and k, KV append, and grouped-query causal
// attention of the call's m rows over the layer's cache, split over the context.
//
// Cache layout of one layer (elements of the cache type, stride = max_pos rounded up to 64):
//   K [kv head][position 0..stride)[head_dim]   (rotated keys, one 2*dh- or 4*dh-byte row per position)
//   V [kv head][head_dim][position 0..stride)   (transposed, so that 8 consecutive positions of one
//                                                dimension are one 128-bit load: the MFMA operand of P.V)
//
// Work item (kv head g, split s): cache positions [s*C, min((s+1)*C, pos0)) of head g (none in the last split, where the
// call's own rows are an item of their own); the last split also
// takes the call's own m rows (rotated, rounded to the cache type, appended to the cache, attended to under
// the causal mask).  All G*m query rows of the group are processed against each K/V element while it is in
// registers or LDS, so the cache is read once.  An item writes one unnormalised partial (o[dh], max, sum)
// per query row; a second, small kernel folds the partials of each row (in a fixed order:
// results are reproducible) and packs the result as the activation block of the Wo GEMM; an item that is its head's
// only one writes that block itself.  There is no
// fence or atomic inside either kernel: the kernel boundary orders them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_launch.h"

namespace ad {

// ---------------------------------------------------------------------------------------------------
// 16-bit cache: MFMA kernel, one wavefront per block of 32 cached positions
// ---------------------------------------------------------------------------------------------------
// The products are those of the fused kernel's attention phase (ad_attention_device.h): S^T = K q^T with the rows of the
// two score tiles assigned to keys so that a lane ends up with 8 consecutive keys of its query row, which is the B operand
// layout of O^T = V^T P^T, K and V^T loaded from the cache straight into operand registers.  Query rows fill all 16
// columns of a tile and their hi and lo parts are two operands (not two halves of the columns), so no score, exponential
// or output is computed twice.  Wavefront w takes blocks w, w + 4, ... of the item under an online softmax (its next K is
// requested as soon as the scores are formed, its next V after the second product); the last wavefront of the last item
// (an item without cached positions, where that leaves one item per compute unit; else the one that holds the end of the
// cache) takes the call's own rows as one more block.  The four wavefronts' results meet in LDS.
//
// An item is a chain of dependent steps, whatever its size, so what counts is its length and how many run at once (a layer's
// cache at context 9203 is read in 6 us).  Layer step of the 8B shape, one layer over and over, against the kernel this replaces (hi and lo parts in the
// two halves of a tile's columns, two wavefronts per block, every item 128 positions): context 9203, 8 rows 142.8 -> 119 us, 1
// row 106.8 -> 100.7; 4096, 4 rows 105.4 -> 102.2; 13B shape, 4096, 8 rows 179.9 -> 171.5.  RT row
// tiles per wavefront, NRH wavefronts per block of keys (each with RT tiles of its own), up to 16 * RT * NRH query rows per pass.
template <int DH, int RT, int NRH>
struct AttnDecLds {
    static constexpr int RP = RT * NRH * 16;
    static constexpr int PD = DH / RT;                     // dimensions folded at a time
    bf16x8 qb[RT * NRH * (DH / 32) * 2 * 64];              // [row tile][k-step][hi, lo][lane]
    uint16_t knew[8 * DH];                                 // the call's own K rows, cache type: [row][dim]
    uint16_t vnewT[DH * 8];                                // the call's own V rows, transposed: [dim][row]
    float mx[4][RP], sum[4][RP];
    float part[4][RP][PD + 4];                             // rows padded to 16 bytes for 128-bit LDS stores
};

// inputs k, k + 1 (k even: the pair is one word) of token t in the packed input of the Wo projection
template <bool F16>
__device__ __forceinline__ void store_act_pair(const AttnArgs &a, int k, int t, float v0, float v1) {
    uint16_t h0, l0, h1, l1;
    split16<F16>(v0, h0, l0);
    split16<F16>(v1, h1, l1);
    *(uint32_t *)((uint16_t *)a.Bo + act_index(k, t, a.Bo_KT)) = (uint32_t)h0 | (uint32_t)h1 << 16;
    *(uint32_t *)((uint16_t *)a.Bo + act_index(k, 8 + t, a.Bo_KT)) = (uint32_t)l0 | (uint32_t)l1 << 16;
}

template <int DH, bool F16, int RT, int NRH>
__global__ void __launch_bounds__(256 * NRH, RT == 1 ? 2 : 1) k_attn_dec(AttnArgs a) {
    warm_kernel_args<sizeof(AttnArgs)>();
    constexpr int KS = DH / 32, DT = DH / 16, half = DH / 2, PR = DH + 2, RP = RT * NRH * 16, NTH = 256 * NRH;
    constexpr float kPScale = F16 ? 1024.0f : 1.0f;        // keeps small probabilities out of fp16's subnormals
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    AttnDecLds<DH, RT, NRH> &L = *reinterpret_cast<AttnDecLds<DH, RT, NRH> *>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) & 3, n = lane & 15, gq = lane >> 4;
    const int row_w = (tid >> 8) * RT * 16;                // this wavefront's first row of a pass
    const int G = a.G, R = a.R;
    const int item = blockIdx.x, g = div_small(item, a.mul_S), s = item - g * a.S;
    const int c0 = s * a.C, c1 = (c0 + a.C < a.pos0) ? c0 + a.C : a.pos0;
    const int nc = (c1 > c0) ? c1 - c0 : 0, nbc = (nc + 31) / 32;       // (none in an item of the own rows alone: c0 >= pos0)
    const bool last = (s == a.S - 1);
    uint16_t *Kg = (uint16_t *)a.Kc + (size_t)g * a.stride * DH;
    uint16_t *Vg = (uint16_t *)a.Vc + (size_t)g * DH * a.stride;
    const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};

    // (addressed as a uniform pointer plus a 32-bit byte offset per lane: one register per load instead of two)
    bf16x8 k[2][KS], v[DT];
    auto load_k = [&](int b) {
#pragma unroll
        for (int aa = 0; aa < 2; ++aa) {
            int key = c0 + b * 32 + 8 * (n >> 2) + 4 * aa + (n & 3);
            if (key > a.pos0 - 1) key = a.pos0 - 1;         // dead positions are masked at use; stay in live memory
            const unsigned off = (unsigned)key * (DH * 2u) + gq * 16u;
#pragma unroll
            for (int j = 0; j < KS; ++j) k[aa][j] = *(const bf16x8 *)((const char *)(Kg + j * 32) + off);
        }
    };
    auto load_v = [&](int b) {
        const unsigned off = ((unsigned)n * (unsigned)a.stride + (unsigned)(c0 + b * 32 + gq * 8)) * 2u;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) v[dt] = *(const bf16x8 *)((const char *)(Vg + (size_t)dt * 16 * a.stride) + off);
    };

    for (int r0 = 0; r0 < R; r0 += RP) {
        const int nr = (R - r0 < RP) ? R - r0 : RP;
        // this wavefront's first cached block goes in flight first: it does not depend on the queries
        if (wave < nbc && row_w < nr) {
            load_k(wave);
            load_v(wave);
        }
        if (last && r0 == 0) {
            // the call's own rows: rotate k, round to the cache type, append to the cache, keep a copy in LDS (from the last thread
            // down: the first ones have the queries)
            for (int idx = NTH - 1 - tid; idx < a.m * half; idx += NTH) {
                const int t = idx / half, i = idx % half;
                const float *kp = a.qkv + (size_t)t * a.ld + (size_t)a.Hq * DH + (size_t)g * DH;
                const float *vp = kp + (size_t)a.Hkv * DH;
                const float c = a.rope[(t * half + i) * 2], sn = a.rope[(t * half + i) * 2 + 1];
                const float x = kp[i], y = kp[i + half];
                const uint16_t k0 = to16<F16>(x * c - y * sn), k1 = to16<F16>(x * sn + y * c);
                const uint16_t v0 = to16<F16>(vp[i]), v1 = to16<F16>(vp[i + half]);
                L.knew[t * DH + i] = k0;
                L.knew[t * DH + i + half] = k1;
                L.vnewT[i * 8 + t] = v0;
                L.vnewT[(i + half) * 8 + t] = v1;
                const size_t p = (size_t)(a.pos0 + t);
                Kg[p * DH + i] = k0;
                Kg[p * DH + i + half] = k1;
                Vg[(size_t)i * a.stride + p] = v0;
                Vg[(size_t)(i + half) * a.stride + p] = v1;
            }
        }
        // queries: rotate, scale, split hi/lo, store in operand order; a thread takes 4 dimensions of each half of a row
        for (int idx = tid; idx < nr * (half / 4); idx += NTH) {
            const int rr = idx / (half / 4), i = (idx % (half / 4)) * 4, r = r0 + rr;
            const int t = div_small(r, a.mul_G), hq = g * G + (r - t * G);
            const float *qp = a.qkv + (size_t)t * a.ld + (size_t)hq * DH + i;
            const float *rp = a.rope + ((size_t)t * half + i) * 2;
            const f32x4 x = *(const f32x4 *)qp, y = *(const f32x4 *)(qp + half);
            const f32x4 ra = *(const f32x4 *)rp, rb = *(const f32x4 *)(rp + 4);
            u16x4 h0, l0, h1, l1;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = e < 2 ? ra[2 * e] : rb[2 * e - 4], sn = e < 2 ? ra[2 * e + 1] : rb[2 * e - 3];
                uint16_t hi, lo;
                split16<F16>((x[e] * c - y[e] * sn) * a.scale, hi, lo);
                h0[e] = hi;
                l0[e] = lo;
                split16<F16>((x[e] * sn + y[e] * c) * a.scale, hi, lo);
                h1[e] = hi;
                l1[e] = lo;
            }
            auto put = [&](int d, int plane, u16x4 w) {
                *(u16x4 *)((uint16_t *)&L.qb[(((rr >> 4) * KS + (d >> 5)) * 2 + plane) * 64 + (rr & 15) + 16 * ((d & 31) >> 3)] + (d & 7)) = w;
            };
            put(i, 0, h0);
            put(i, 1, l0);
            put(i + half, 0, h1);
            put(i + half, 1, l1);
        }
        __syncthreads();

        f32x4 o[RT][DT];
        float mx[RT], sum[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            mx[i] = -INFINITY;
            sum[i] = 0.f;
#pragma unroll
            for (int d = 0; d < DT; ++d) o[i][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        // one block of 32 keys, in k and v: `live` of them from the block's start (IS_NEW: the call's own rows, causal)
        auto block = [&](auto is_new, int live, auto after_scores) {
            constexpr bool IS_NEW = decltype(is_new)::value;
            f32x4 sc[RT][2];
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                sc[i][0] = sc[i][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (row_w + i * 16 < nr) {
#pragma unroll
                    for (int j = 0; j < KS; ++j)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const bf16x8 q = L.qb[(((row_w / 16 + i) * KS + j) * 2 + p) * 64 + lane];
                            sc[i][0] = mma16<F16>(k[0][j], q, sc[i][0]);
                            sc[i][1] = mma16<F16>(k[1][j], q, sc[i][1]);
                        }
                }
            }
            after_scores();
            bf16x8 ph[RT], pl[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                if (row_w + i * 16 >= nr) continue;
                const int t_row = IS_NEW ? div_small(r0 + row_w + i * 16 + n, a.mul_G) : 0;
                float w[8], bm = -INFINITY;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    w[c] = sc[i][c >> 2][c & 3];
                    const int key = gq * 8 + c;
                    if (IS_NEW ? (key >= a.m || key > t_row) : key >= live) w[c] = -INFINITY;
                    bm = fmaxf(bm, w[c]);
                }
                bm = max_rows(bm);
                const float nm = fmaxf(mx[i], bm), ref = softmax_ref(nm);
                const float alpha = __expf(mx[i] - ref);
                mx[i] = nm;
                float add = 0.f;
                u16x8 h8, l8;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float p = __expf(w[c] - ref);
                    add += p;
                    uint16_t hi, lo;
                    split16<F16>(p * kPScale, hi, lo);
                    h8[c] = hi;
                    l8[c] = lo;
                }
                ph[i] = __builtin_bit_cast(bf16x8, h8);
                pl[i] = __builtin_bit_cast(bf16x8, l8);
                sum[i] = sum[i] * alpha + add;
                if (!__all(alpha == 1.0f)) {
#pragma unroll
                    for (int d = 0; d < DT; ++d) o[i][d] *= alpha;
                }
            }
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                if (row_w + i * 16 >= nr) continue;
#pragma unroll
                for (int d = 0; d < DT; ++d) {
                    o[i][d] = mma16<F16>(v[d], ph[i], o[i][d]);
                    o[i][d] = mma16<F16>(v[d], pl[i], o[i][d]);
                }
            }
        };
        for (int b = wave; b < nbc && row_w < nr; b += 4) {
            const int live = nc - b * 32;
            if (live < 32) {                                // ragged end of the cache: dead positions contribute nothing
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (gq * 8 + e >= live) v[dt][e] = 0;
            }
            block(std::false_type{}, live, [&]() { if (b + 4 < nbc) load_k(b + 4); });
            if (b + 4 < nbc) load_v(b + 4);
        }
        if (last && wave == 3 && row_w < nr) {
#pragma unroll
            for (int aa = 0; aa < 2; ++aa) {
                const int key = 8 * (n >> 2) + 4 * aa + (n & 3);
#pragma unroll
                for (int j = 0; j < KS; ++j) k[aa][j] = (key < a.m) ? *(const bf16x8 *)(L.knew + key * DH + j * 32 + gq * 8) : zero;
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                // keys gq * 8 .. + 7 of dimension dt * 16 + n: only the first lane group has live keys
                bf16x8 cv = (gq == 0) ? *(const bf16x8 *)(L.vnewT + (dt * 16 + n) * 8) : zero;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e >= a.m) cv[e] = 0;
                v[dt] = cv;
            }
            block(std::true_type{}, 0, []() {});
        }
        // lane (n, gq): row n of a tile, dimensions d*16 + gq*4 .. +3.  The wavefronts' results are folded in wavefront order, PD
        // dimensions at a time: a thread takes two neighbouring dimensions of a row and derives the wavefronts' weights itself.
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const float den = sum_rows(sum[i]);
            if (gq == 0) {
                L.mx[wave][row_w + i * 16 + n] = mx[i];
                L.sum[wave][row_w + i * 16 + n] = den;
            }
        }
        constexpr int PD = AttnDecLds<DH, RT, NRH>::PD;
#pragma unroll
        for (int h = 0; h < RT; ++h) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int d = 0; d < PD / 16; ++d)
                    if (row_w + i * 16 + n < nr) *(f32x4 *)&L.part[wave][row_w + i * 16 + n][d * 16 + gq * 4] = o[i][h * (PD / 16) + d] * (1.0f / kPScale);
            __syncthreads();
            for (int idx = tid; idx < nr * (PD / 2); idx += NTH) {
                const int rr = idx / (PD / 2), e = (idx % (PD / 2)) * 2;
                float mp[4], M = -INFINITY, sm[4], den = 0.f;
                f32x2 x[4], num = {0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    mp[w] = L.mx[w][rr];
                    sm[w] = L.sum[w][rr];
                    x[w] = *(const f32x2 *)&L.part[w][rr][e];
                    M = fmaxf(M, mp[w]);
                }
                const float ref = softmax_ref(M);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float f = __expf(mp[w] - ref);    // a wavefront without keys: exp(-inf) = 0, of sums that are 0
                    den += f * sm[w];
                    num[0] += f * x[w][0];
                    num[1] += f * x[w][1];
                }
                if (a.S == 1) {                             // nothing to fold: the output itself, packed for the Wo GEMM
                    const int r = r0 + rr, t = div_small(r, a.mul_G), kk = (g * G + (r - t * G)) * DH + h * PD + e;
                    store_act_pair<F16>(a, kk, t, num[0] / den, num[1] / den);
                    continue;
                }
                float *out = a.part + (((size_t)g * a.S + s) * R + (r0 + rr)) * PR;
                *(f32x2 *)(out + h * PD + e) = num;
                if (h == 0 && e == 0) *(f32x2 *)(out + DH) = (f32x2){M, den};
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// fp32 cache: vector-ALU kernel (the model is small)
// ---------------------------------------------------------------------------------------------------
// An item is a chain of instructions and three barriers.  K and V go from the cache into registers, once for all query rows and before
// anything else: a thread holds 16 dimensions of one key (DH / 16 neighbouring lanes have the rest) and 16 keys of one dimension
// (512 / DH neighbouring lanes have the rest); dot products and sums are finished by moves between lanes.  Against the kernel
// before it (1024 threads, K and V through LDS, all query rows of a head in one workgroup): 4 heads of 64, context 47, 1 row 6.1 ->
// 4.1 us; 2 kv heads, context 500, 12 query rows per head 14.3 -> 4.7 (10.2 with all rows in one workgroup).
constexpr int kValuThreads = 512;
constexpr int kValuMaxRows = 32;
constexpr int valu_chunk(int dh) { return kValuThreads * 16 / dh; }      // cached positions per item: a key per DH / 16 threads

template <int DH>
__global__ void __launch_bounds__(kValuThreads, 2) k_attn_valu(AttnArgs a) {
    warm_kernel_args<sizeof(AttnArgs)>();
    constexpr int C = valu_chunk(DH), LK = DH / 16, TE = kValuThreads / DH, half = DH / 2, MAXK = C + 8, PR = DH + 2;
    __shared__ __attribute__((aligned(16))) float qs[kValuMaxRows][DH], sc[kValuMaxRows][MAXK], knew[8][DH], vnew[8][DH];
    __shared__ float st[kValuMaxRows][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int G = a.G, R = a.R;
    // x / d for any x: the rounded-up reciprocal is never too small and, below 2^32, at most one too large (models of 32767 query heads
    // per kv head and more have rows past the numbers that it is exact for)
    auto quotient = [](int x, int d, unsigned mul) {
        const int q = div_small(x, mul);
        return q * d > x ? q - 1 : q;
    };
    const int item = blockIdx.x, g = quotient(item, a.S, a.mul_S), s = item - g * a.S;
    const int c0 = s * C, c1 = (c0 + C < a.pos0) ? c0 + C : a.pos0;
    const int nc = (c1 > c0) ? c1 - c0 : 0;
    const bool last = (s == a.S - 1);
    const int r_first = blockIdx.y * a.rows_wg, r_end = r_first + a.rows_wg < R ? r_first + a.rows_wg : R;     // this workgroup's query rows
    float *Kg = (float *)a.Kc + (size_t)g * a.stride * DH, *Vg = (float *)a.Vc + (size_t)g * DH * a.stride;
    const int key = tid / LK, d0 = (tid % LK) * 16;             // products with K: key, first dimension
    const int e = tid / TE, part = tid % TE;                    // products with V: dimension, keys (i * TE + part) * 4 .. + 3
    f32x4 k[4], v[4];
    {
        const float *kp = Kg + (size_t)(key < nc ? c0 + key : 0) * DH + d0;     // keys past the item's are masked at use
#pragma unroll
        for (int i = 0; i < 4; ++i) k[i] = *(const f32x4 *)(kp + i * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = (i * TE + part) * 4;                  // (a group that starts before the item's end lies inside the cache row)
            v[i] = *(const f32x4 *)(Vg + (size_t)e * a.stride + (j < nc ? c0 + j : 0));
        }
    }
    if (last) {
        // the call's own rows: rotate k, append to the cache, keep a copy in LDS
        for (int idx = tid; idx < a.m * half; idx += kValuThreads) {
            const int t = idx / half, i = idx % half;
            const float *kp = a.qkv + (size_t)t * a.ld + (size_t)a.Hq * DH + (size_t)g * DH;
            const float *vp = kp + (size_t)a.Hkv * DH;
            const float c = a.rope[(t * half + i) * 2], sn = a.rope[(t * half + i) * 2 + 1];
            const float x = kp[i], y = kp[i + half];
            const float k0 = x * c - y * sn, k1 = x * sn + y * c;
            const float v0 = vp[i], v1 = vp[i + half];
            knew[t][i] = k0;
            knew[t][i + half] = k1;
            vnew[t][i] = v0;
            vnew[t][i + half] = v1;
            if (blockIdx.y == 0) {
                const size_t p = (size_t)(a.pos0 + t);
                Kg[p * DH + i] = k0;
                Kg[p * DH + i + half] = k1;
                Vg[(size_t)i * a.stride + p] = v0;
                Vg[(size_t)(i + half) * a.stride + p] = v1;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if ((i * TE + part) * 4 + c >= nc) v[i][c] = 0.f;   // dead positions may hold anything
    auto sum_lanes = [](float x, int n) {                       // over n = 4 or 8 neighbouring lanes
        x += dpp<0xB1>(x);
        x += dpp<0x4E>(x);
        if (n == 8) x += dpp<0x141>(x);
        return x;
    };
    for (int r0 = r_first; r0 < r_end; r0 += kValuMaxRows) {
        const int nr = (r_end - r0 < kValuMaxRows) ? r_end - r0 : kValuMaxRows;
        for (int idx = tid; idx < nr * half; idx += kValuThreads) {
            const int rr = idx / half, i = idx % half, r = r0 + rr, t = quotient(r, G, a.mul_G), hq = g * G + (r - t * G);
            const float *qp = a.qkv + (size_t)t * a.ld + (size_t)hq * DH;
            const float c = a.rope[(t * half + i) * 2], sn = a.rope[(t * half + i) * 2 + 1];
            const float x = qp[i], y = qp[i + half];
            qs[rr][i] = (x * c - y * sn) * a.scale;
            qs[rr][i + half] = (x * sn + y * c) * a.scale;
        }
        __syncthreads();
        auto dot = [&](int rr, const f32x4 (&kk)[4]) {
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 q = *(const f32x4 *)&qs[rr][d0 + i * 4];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc += q[c] * kk[i][c];
            }
            return sum_lanes(acc, LK);
        };
        for (int rr = 0; rr < nr; ++rr) {
            const float x = dot(rr, k);
            if (tid % LK == 0) sc[rr][key] = key < nc ? x : -INFINITY;
        }
        if (last && key < 8) {                                  // (whole groups of lanes that add up; keys past the call's are masked)
            f32x4 kk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) kk[i] = *(const f32x4 *)&knew[key][d0 + i * 4];
            for (int rr = 0; rr < nr; ++rr) {
                const float x = dot(rr, kk);
                const int t = quotient(r0 + rr, G, a.mul_G);    // causal mask among the call's own rows
                if (tid % LK == 0) sc[rr][C + key] = key < a.m && key <= t ? x : -INFINITY;
            }
        }
        __syncthreads();
        for (int rr = wave; rr < nr; rr += kValuThreads / 64) {
            constexpr int NV = (MAXK + 63) / 64;
            float x[NV], mx = -INFINITY, sum = 0.f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int j = i * 64 + lane;
                x[i] = j < (last ? MAXK : C) ? sc[rr][j] : -INFINITY;
                mx = fmaxf(mx, x[i]);
            }
            mx = max64(mx);
            const float ref = softmax_ref(mx);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const float p = __expf(x[i] - ref);
                if (i * 64 + lane < MAXK) sc[rr][i * 64 + lane] = p;
                sum += p;
            }
            sum = sum64(sum);
            if (lane == 0) {
                st[rr][0] = mx;
                st[rr][1] = sum;
            }
        }
        __syncthreads();
        for (int rr = 0; rr < nr; ++rr) {
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 p = *(const f32x4 *)&sc[rr][(i * TE + part) * 4];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc += p[c] * v[i][c];
            }
            if (last)
                for (int t = part; t < a.m; t += TE) acc += sc[rr][C + t] * vnew[t][e];
            acc = sum_lanes(acc, TE);
            if (part == 0) {
                if (a.S == 1) {                                 // nothing to fold: the output itself, packed for the Wo GEMM
                    const int r = r0 + rr, t = quotient(r, G, a.mul_G);
                    store_act<false>(a.Bo, a.Bo_KT, (g * G + (r - t * G)) * DH + e, t, acc / st[rr][1]);
                } else {
                    float *pr = a.part + (((size_t)g * a.S + s) * R + (r0 + rr)) * PR;
                    pr[e] = acc;
                    if (e == 0) {
                        pr[DH] = st[rr][0];
                        pr[DH + 1] = st[rr][1];
                    }
                }
            }
        }
        if (r0 + kValuMaxRows < r_end) __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------
// fold the splits of every query row, in split order, and pack the result for the Wo GEMM
// ---------------------------------------------------------------------------------------------------
// One workgroup per query row: DH / 2 threads (two neighbouring dimensions each) times NG groups, a group taking every NG-th
// split, KB of them at a time.  A thread loads its splits' (max, sum) itself, the same address for its whole group, so that
// nothing but the groups' results crosses threads.  The kernel is a chain of instructions more than a move of data: with one
// wavefront per row (and up to 32 splits in flight, the weights handed around by shuffles) the layer step of the 8B shape took
// 92.4 us against 91.2 now (1 row, context 4096), 113.5 / 112.0 (8 rows, 9203), that of the 13B shape 129.8 / 128.3 (2 rows, 777).
template <int DH, bool F16>
__global__ void __launch_bounds__(256) k_attn_combine(const float *partials, void *Bo, uint64_t s_r, uint64_t g_kt, uint64_t mul_r_g) {
    AttnArgs a;
    a.Bo = Bo; a.R = (int)(s_r >> 32); a.G = (int)g_kt; a.Bo_KT = (int)(g_kt >> 32); a.mul_R = (unsigned)mul_r_g; a.mul_G = (unsigned)(mul_r_g >> 32);
    constexpr int PR = DH + 2, TG = DH / 2, NG = 256 / TG, KB = 8;
    __shared__ float st[NG][2];
    __shared__ f32x2 part[NG][TG];
    const int tid = threadIdx.x, grp = TG == 64 ? __builtin_amdgcn_readfirstlane(tid / TG) : tid / TG, e = 2 * (tid % TG), S = (int)s_r;
    const int row = blockIdx.x, g = div_small(row, a.mul_R), r = row - g * a.R, t = div_small(r, a.mul_G), hq = g * a.G + (r - t * a.G);
    const float *base = partials + ((size_t)g * S * a.R + r) * PR;
    float M = -INFINITY, den = 0.f;
    f32x2 o = {0.f, 0.f};
    for (int s0 = grp; s0 < S; s0 += NG * KB) {
        f32x2 v[KB], ms[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) {                          // splits past the end repeat the group's first (weight 0)
            const int s = s0 + k * NG;
            // (32 bits count rows of partials, not their floats: an fp32 cache's splits grow with the context)
            const float *p = base + (size_t)((unsigned)(s < S ? s : s0) * (unsigned)a.R) * PR;
            ms[k] = *(const f32x2 *)(p + DH);
            v[k] = *(const f32x2 *)(p + e);
        }
        float nm = M;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (s0 + k * NG >= S) ms[k] = (f32x2){-INFINITY, 0.f};
            nm = fmaxf(nm, ms[k][0]);
        }
        const float ref = softmax_ref(nm), alpha = __expf(M - ref);
        M = nm;
        den *= alpha;
        o *= alpha;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const float w = __expf(ms[k][0] - ref);
            den += w * ms[k][1];
            o[0] += w * v[k][0];
            o[1] += w * v[k][1];
        }
    }
    part[grp][tid % TG] = o;
    if (e == 0) {
        st[grp][0] = M;
        st[grp][1] = den;
    }
    __syncthreads();
    if (tid >= TG) return;
    float m = -INFINITY, d = 0.f;
    f32x2 y = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NG; ++i) m = fmaxf(m, st[i][0]);
    const float ref = softmax_ref(m);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const float w = __expf(st[i][0] - ref);                 // a group without splits: exp(-inf) = 0
        d += w * st[i][1];
        y += w * part[i][tid];
    }
    store_act_pair<F16>(a, hq * DH + e, t, y[0] / d, y[1] / d);
}

// ---------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------
int attn_chunk(int kv_elem, int dh) { return kv_elem != kElemF32 ? 128 : valu_chunk(dh); }

template <int DH>
static int launch_valu(const AttnArgs &a, const LaunchCtx &c) {
    // A head's query rows are dealt to several workgroups, down to two each, while there are compute units to spare (each reads the
    // head's positions for itself).
    AttnArgs b = a;
    const int spare = c.n_wg / (a.Hkv * a.S), most = (a.R + 1) / 2;
    const int nz = spare < 1 ? 1 : spare < most ? spare : most;
    b.rows_wg = (a.R + nz - 1) / nz;
    return launch<k_attn_valu<DH>>(c, dim3(a.Hkv * a.S, (a.R + b.rows_wg - 1) / b.rows_wg), dim3(kValuThreads), 0, b);
}

template <int DH, bool F16, int RT, int NRH>
static int launch_dec_as(const AttnArgs &a, const LaunchCtx &c) {
    const size_t lds = sizeof(AttnDecLds<DH, RT, NRH>);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_attn_dec<DH, F16, RT, NRH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    return launch<k_attn_dec<DH, F16, RT, NRH>>(c, dim3(a.Hkv * a.S), dim3(256 * NRH), lds, a);
}

// More than 16 query rows: two wavefronts per block of keys, a row tile each, while an item is one block per wavefront (the chain
// through an item is what counts then); else one wavefront with both tiles (and all the registers that takes: held to 256 of
// them it spilled 25, and the 8B shape's step of 8 rows at context 9203 took 111.0 us and not 106.1).  Layer step of the 8B shape,
// 5 / 8 rows, two wavefronts against one: context 300 93.5 / 99.6 us, 94.0 / 100.2; 4096 97.6 / 105.1, 98.4 / 105.5; 6000 (two
// blocks per wavefront) 98.1 / 104.5, 97.6 / 104.1; 9203 (three) 101.8 / 108.3, 99.9 / 106.6.
template <int DH, bool F16>
static int launch_dec(const AttnArgs &a, const LaunchCtx &c) {
    if (a.R <= 16) return launch_dec_as<DH, F16, 1, 1>(a, c);
    if (a.C <= attn_chunk(a.kv_elem, a.dh) || a.S == 1) return launch_dec_as<DH, F16, 1, 2>(a, c);
    return launch_dec_as<DH, F16, 2, 1>(a, c);
}

// Positions per item for a stand-alone launch, k times the smallest item: one item per compute unit if k = 4 is enough for
// that, else two.  (An item that shares its compute unit runs slower, but a chain of many blocks is longer still.)
// Contexts up to two items' length get one item per kv head, which writes the attention output itself.  Layer of a stretch, two
// items and the fold against one item, context 256, 1 / 8 rows: 8B shape 94.3 -> 92.1 / 109.3 -> 109.0 us, 13B 132.7 -> 130.0 /
// 159.2 -> 156.7, 2 kv heads of 64 dimensions 32.7 -> 29.2 / 36.5 -> 33.1; slower only with 64 query rows on a lone kv head of 128
// (1 row 40.0 -> 37.4, 8 rows 56.3 -> 58.8).  Three items in one: 8B, 4 rows 99.6 -> 98.9, 8 rows 110.8 -> 115.8.
// Measured, layer step, one layer over and over: 8B shape, 1 row, context 9203: k = 3 (192 items) 100.7 us, k = 2 (288) 103.2, k = 1 (576) 107.5;
// 13B shape (40 kv heads), 1 row, context 4096: k = 3 (440 items) 143.2 us, k = 5 (280) 149.7, k = 2 (640) 147.1.
int attn_chunk_for(int kv_elem, int dh, int n_kv_heads, int pos0, int n_wg) {
    const int c = attn_chunk(kv_elem, dh);
    if (kv_elem == kElemF32) return c;
    if (pos0 <= 2 * c) return pos0 <= c ? c : 2 * c;       // one item per kv head: nothing to fold, one kernel less
    auto items = [&](int k) { return (long)n_kv_heads * ((pos0 + (long)k * c - 1) / ((long)k * c)); };
    for (int k = 1; k <= 4; ++k)
        if (items(k) <= n_wg) return k * c;
    for (int k = 2;; ++k)                                  // ends: with one item per kv head at the latest
        if (items(k) <= 2L * n_wg || items(k) <= n_kv_heads) return k * c;
}

// The own rows are a second chain (rotation, append, one more block) behind the last item's own: on a compute unit of their own if
// there is one to spare.  Layer step of the 8B shape, 1 row, context 2048 88.1 -> 86.0 us, 8 rows 103.1 -> 100.8, 300 and 1201 alike;
// with 264 items for 256 compute units (context 4096) 88.7 -> 89.3.
bool attn_own_item(int kv_elem, int n_kv_heads, int S, int n_wg) {
    return kv_elem != kElemF32 && S > 1 && (long)n_kv_heads * (S + 1) <= n_wg;
}

template <int DH, bool F16>
static int launch_combine(const AttnArgs &a, dim3 rows, const LaunchCtx &c) {
    return launch<k_attn_combine<DH, F16>>(c, rows, dim3(256), 0, a.part, a.Bo, two(a.S, a.R), two(a.G, a.Bo_KT), two((int)a.mul_R, (int)a.mul_G));
}

int launch_attn(const AttnArgs &a, const LaunchCtx &c) {
    int rc;
    if (a.kv_elem == kElemBF16) {
        if (a.dh == 128) rc = launch_dec<128, false>(a, c);
        else if (a.dh == 64) rc = launch_dec<64, false>(a, c);
        else return (int)hipErrorInvalidValue;
    } else if (a.kv_elem == kElemF16) {
        if (a.dh == 128) rc = launch_dec<128, true>(a, c);
        else if (a.dh == 64) rc = launch_dec<64, true>(a, c);
        else return (int)hipErrorInvalidValue;
    } else {
        if (a.dh == 128) rc = launch_valu<128>(a, c);
        else if (a.dh == 64) rc = launch_valu<64>(a, c);
        else return (int)hipErrorInvalidValue;
    }
    if (rc || a.S == 1) return rc;
    const dim3 rows(a.Hq * a.m);
    if (a.kv_elem == kElemF16) return a.dh == 128 ? launch_combine<128, true>(a, rows, c) : launch_combine<64, true>(a, rows, c);
    return a.dh == 128 ? launch_combine<128, false>(a, rows, c) : launch_combine<64, false>(a, rows, c);
}

}  // namespace ad
