// The prompt pass: up to kPromptRows tokens through a decoder layer at once (16-bit models).  A layer step takes at most 8
// rows and reads the layer's weights for them; here a weight tile that has reached the chip is multiplied by all the
// tokens of a workgroup, and the pass is bound by the matrix cores instead of by memory.
//
// The arithmetic is the layer step's: activations are split into 16-bit hi and lo parts, both are multiplied, sums are
// fp32; K and V are rounded to the cache type when they are stored and attention reads the stored values.
//
// Per layer: k_prompt_gemm (q, k, v) -> k_prompt_qkv (rotation, KV append, query tiles) -> k_prompt_attn ->
// k_prompt_gemm (Wo) -> k_prompt_rows (residual, RMSNorm, tiles) -> k_prompt_gemm (gate/up, SwiGLU) ->
// k_prompt_gemm (down) -> k_prompt_rows.  The last layer is its K and V alone.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ad_device.h"
#include "ad_internal.h"
#include "ad_prompt.h"
#include "ad_prompt_layout.h"

namespace ad {

namespace {

// 16-byte unit of token t, inputs k .. k + 7 (k a multiple of 8), in activation tiles with KT k-steps (plane 0 = hi)
__device__ __forceinline__ size_t act_unit(int t, int k, int KT, int plane) {
    return (((size_t)(t >> 4) * KT + (k >> 5)) * 2 + plane) * 64 + (t & 15) + 16 * ((k & 31) >> 3);
}

// ---------------------------------------------------------------------------------------------------
// projections
// ---------------------------------------------------------------------------------------------------
// A workgroup of NWR x NWT wavefronts computes BR = NWR * WR row tiles x BT = NWT * WT token tiles; a wavefront holds
// WR x WT accumulators.  Both operands lie in memory in MFMA operand order, so tiles are copied as they are and every LDS
// access is 64 consecutive 16-byte units: no bank conflicts, no address arithmetic.
//
// The accumulators are emptied into a second set every few k-steps, each at its own turn: one long chain of fp32 additions is off by
// 5.7e-7 of the result at K = 4096 and 1.1e-6 at 14336.  Squared, the error is 4.7e-15 * n (n + 1) / 2 for every chain of n k-steps (two products, each
// rounded several times), 6.7e-16 times the k-steps in the sum for every addition to it, and 8e-16 times those in the pieces for
// every piece added, over the k-steps of the product (fitted to 414 products of 1024 to 14336 inputs, within 3 %).  So short pieces are emptied every kFlush
// k-steps, and those of more than kLongPiece (ad_prompt_layout.h), whose sums are longer, every kFlushLong; a tail that is no multiple of it lengthens the last chain.
constexpr int kFlush = 4, kFlushLong = 8;
enum { PG_PART = 0, PG_SWIGLU = 1 };

// Which tile and piece this workgroup has.  Workgroups are dealt to the 8 XCDs in turn: each XCD gets a contiguous run
// of (piece, row block, token block), so that the workgroups that share weights share an L2.  Tiles from g.n_full on are dealt as
// two halves of their rows (half 0 or 1; else -1), a workgroup each.
struct PromptTile { int rb, tb, piece, half; };
__device__ __forceinline__ PromptTile prompt_tile(const PromptGemm &g) {
    const int tiles = g.n_rb * g.n_tb * g.n_split;
    const bool halves = (int)blockIdx.x >= g.n_full;
    const int n = halves ? 2 * (tiles - g.n_full) : g.n_full, b = (int)blockIdx.x - (halves ? g.n_full : 0);
    const int q8 = n >> 3, r8 = n & 7, xcd = b & 7;
    const int id = xcd * q8 + (xcd < r8 ? xcd : r8) + (b >> 3);
    const int tile = halves ? g.n_full + (id >> 1) : id;
    PromptTile t;
    t.half = halves ? id & 1 : -1;
    t.tb = tile % g.n_tb;
    const int rest = tile / g.n_tb;
    t.rb = rest % g.n_rb;
    t.piece = rest / g.n_rb;
    return t;
}

template <int WR, int WT>
struct PromptAcc {
    f32x4 acc[WR][WT], sum[WR][WT];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) acc[i][j] = sum[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    // empties the accumulators into the sums
    __device__ __forceinline__ void flush() {
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                sum[i][j] += acc[i][j];
                acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
    }
    // the same for those whose turn is k-step s of F: a few at every k-step, so that the additions go by between products
    template <int F>
    __device__ __forceinline__ void flush_some(int s) {
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j)
                if ((i * WT + j) * F / (WR * WT) == s) {
                    sum[i][j] += acc[i][j];
                    acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
                }
    }
    // stores the sums of the tiles rt0 .., tt0 ..; a tile's lane (n, gq) holds token n, rows gq*4 .. +3
    template <bool F16, int EPI>
    __device__ __forceinline__ void store(const PromptGemm &g, int rt0, int tt0, int piece, int lane) const {
        const int n = lane & 15, gq = lane >> 4;
#pragma unroll
        for (int t = 0; t < WT; ++t) {
            const int tok = (tt0 + t) * 16 + n;
            const float scale = (EPI == PG_SWIGLU && tok < g.M) ? g.scale[tok] : 0.f;
#pragma unroll
            for (int r = 0; r < WR; ++r) {
                const int rt = rt0 + r;
                if (EPI == PG_PART) {
                    const int row = rt * 16 + gq * 4;
                    if (tok < g.M && row < g.N) *(f32x4 *)(g.part + ((size_t)piece * g.M + tok) * g.N + row) = sum[r][t];
                } else {
                    // rows 0..7 of a tile are gate, 8..15 up of the same 8 features: the other half sits 32 lanes away.  Both
                    // halves then hold the products of 4 features; the lower one stores their hi parts, the upper the lo parts.
                    u16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float mine = scale * sum[r][t][e], other = __shfl_xor(mine, 32);
                        const float gate = gq < 2 ? mine : other, up = gq < 2 ? other : mine;
                        uint16_t hi, lo;
                        split16<F16>(gate / (1.0f + __expf(-gate)) * up, hi, lo);
                        v[e] = gq < 2 ? hi : lo;
                    }
                    if (tok < g.M && rt < g.NT) {
                        uint16_t *u = (uint16_t *)((bf16x8 *)g.Bnext + act_unit(tok, rt * 8, g.Bnext_KT, gq >> 1));
                        *(u16x4 *)(u + 4 * (gq & 1)) = v;
                    }
                }
            }
        }
    }
};

constexpr int prompt_stage_units(int br, int bt) { return br * 64 + bt * 128; }

// 1 KiB from memory straight into LDS: lane l's 16 bytes go to unit l of dst (the same for all lanes)
__device__ __forceinline__ void copy_to_lds(const void *src, bf16x8 *dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// One workgroup's tile: row tiles rt0 .., token block tb, k-steps of a piece.
//
// Weights and activations are copied from memory into LDS without a way through registers, up to NST k-steps ahead.  A k-step is two
// phases, the products with the hi plane and those with the lo plane; in each the operands of the next phase are read from LDS, one read
// between two products, so that no product waits for LDS.  Between the phases is the step's only barrier: behind it the next stage is
// there and nobody reads this one any more, whose place the copies of k-step s + NST then take, half of them in this lo phase and half in the
// next hi phase, spread between the products (all at once they hold up the products behind them).  ONE: a single phase, for tiles of so few
// products that the reads take longer than a phase of them.
template <int WR, int WT, int NWR, int NWT, int NST, bool F16, int EPI, int F, bool ONE>
__device__ __forceinline__ void prompt_gemm_tile(const PromptGemm &g, int rt0, int tb, int piece, bf16x8 *lds) {
    constexpr int NW = NWR * NWT, BR = WR * NWR, BT = WT * NWT;
    constexpr int SU = prompt_stage_units(BR, BT), UNITS = BR + BT * 2;         // 16-byte units, and KiB, per stage
    constexpr int NC = (UNITS + NW - 1) / NW, NH = ONE ? NC : NC / 2;      // copies of a wavefront per stage, of them in the lo phase
    // Copies of a wavefront that may be in flight at a step's barrier.  The wait counts them, so that copies have to be issued in the
    // order of their stages: no copy moves past the scheduling barriers between phases.
    constexpr int FLY = NC * (NST - 2), FLY0 = NC * (NST - 2) + NH;
    static_assert(FLY0 < 64 && NST >= 3, "the counter of loads in flight has six bits");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % NWR, wt = wave / NWR;
    const int k0 = piece * g.k_per, k1 = k0 + g.k_per < g.KT ? k0 + g.k_per : g.KT;

    const char *src[NC];
    unsigned off[NC];
    int shift[NC], dst[NC];                                     // log2 of the bytes from one k-step to the next; place in a stage
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        int u = wave * NC + i;                                  // 1 KiB of a stage: a weight tile, or a token tile's plane
        if (u > UNITS - 1) u = UNITS - 1;                       // (no more of them: the last one again, to the same place)
        dst[i] = u * 64;
        if (u < BR) {
            int rt = rt0 + u;
            if (rt > g.NT - 1) rt = g.NT - 1;                   // past the last row tile: its products are not stored
            src[i] = (const char *)g.W;
            off[i] = ((unsigned)rt * (unsigned)g.KT * 64u + (unsigned)lane) << 4;
            shift[i] = 10;
        } else {
            const int v = u - BR, last = (g.M + 15) / 16 - 1;
            int tt = tb * BT + (v >> 1);
            if (tt > last) tt = last;                           // past the last token tile: likewise
            src[i] = (const char *)g.B;
            off[i] = ((unsigned)tt * (unsigned)g.KT * 128u + (unsigned)((v & 1) * 64 + lane)) << 4;
            shift[i] = 11;
        }
    }
    const int k_last = k1 - 1;                                  // copies past the piece repeat its last k-step
    auto copy = [&](int stage, int k, int i0, int i1) {
        const int kk = k < k_last ? k : k_last;
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (i >= i0 && i < i1) copy_to_lds(src[i] + (size_t)(off[i] + ((unsigned)kk << shift[i])), lds + stage * SU + dst[i]);
    };
    // waits until no more than n copies are in flight and every read of LDS is done (bits of the immediate: vmcnt 0-3 and 14-15, lgkmcnt
    // 8-11, expcnt 4-6, all ones, is not waited for), then for everyone else
    auto meet = [&](auto n) {
        constexpr int N = decltype(n)::value;
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | (N >> 4 << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    PromptAcc<WR, WT> C;
    C.clear();
    struct Operands { bf16x8 a[WR], hi[WT], lo[WT]; } x, y;
    const int la = wr * WR * 64 + lane, lb = BR * 64 + wt * WT * 128 + lane;
    auto fetch_hi = [&](Operands &o, int stage) {
        const bf16x8 *p = lds + stage * SU;
#pragma unroll
        for (int r = 0; r < WR; ++r) o.a[r] = p[la + r * 64];
#pragma unroll
        for (int t = 0; t < WT; ++t) o.hi[t] = p[lb + t * 128];
    };
    auto fetch_lo = [&](Operands &o, int stage) {
        const bf16x8 *p = lds + stage * SU;
#pragma unroll
        for (int t = 0; t < WT; ++t) o.lo[t] = p[lb + t * 128 + 64];
    };
    auto mma = [&](const bf16x8 (&w)[WR], const bf16x8 (&b)[WT]) {
#pragma unroll
        for (int r = 0; r < WR; ++r)
#pragma unroll
            for (int t = 0; t < WT; ++t) C.acc[r][t] = mma16<F16>(w[r], b[t], C.acc[r][t]);
    };
    // a product, a read of LDS, in turn; then the copies, behind a few products each; then the rest of the products
    auto interleave = [](auto reads, auto copies) {
        constexpr int R = decltype(reads)::value, CP = decltype(copies)::value;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < CP; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, WR * WT, 0);
    };
    const int n_step = k1 - k0;
    int cur = 0, prev = NST - 1;
    // turn: which accumulators the step empties (-1: none)
    auto step = [&](int s, int turn, Operands &now, Operands &next) {
        const int nxt = cur == NST - 1 ? 0 : cur + 1;
        if constexpr (ONE) {
            meet(std::integral_constant<int, FLY>{});
            fetch_hi(next, nxt);
            fetch_lo(next, nxt);
            copy(cur, k0 + s + NST, 0, NC);
            if (turn >= 0) C.template flush_some<F>(turn);
            mma(now.a, now.hi);
            mma(now.a, now.lo);
        } else {
            fetch_lo(now, cur);
            copy(prev, k0 + s + NST - 1, NH, NC);
            if (turn >= 0) C.template flush_some<F>(turn);
            mma(now.a, now.hi);
            interleave(std::integral_constant<int, WT>{}, std::integral_constant<int, NC - NH>{});
            meet(std::integral_constant<int, FLY>{});
            fetch_hi(next, nxt);
            copy(cur, k0 + s + NST, 0, NH);
            mma(now.a, now.lo);
            interleave(std::integral_constant<int, WR + WT>{}, std::integral_constant<int, NH>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        prev = cur;
        cur = nxt;
    };
#pragma unroll
    for (int j = 0; j < NST; ++j) {
        copy(j, k0 + j, 0, j < NST - 1 ? NC : NH);
        __builtin_amdgcn_sched_barrier(0);
    }
    meet(std::integral_constant<int, FLY0>{});
    fetch_hi(x, 0);
    if constexpr (ONE) fetch_lo(x, 0);
    int s = 0;
    for (; s + F <= n_step; s += F) {
#pragma unroll
        for (int j = 0; j < F; j += 2) {
            step(s + j, j, x, y);
            step(s + j + 1, j + 1, y, x);
        }
    }
    for (; s < n_step; ++s) {
        step(s, -1, x, y);
        x = y;
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                         // the copies past the end land before the workgroup's LDS is another's
    C.flush();
    C.template store<F16, EPI>(g, rt0 + wr * WR, tb * BT + wt * WT, piece, lane);
}

// F: k-steps from one emptying of an accumulator to the next.  HALVES: tiles from g.n_full on are workgroups of half the rows.
template <int WR, int WT, int NWR, int NWT, int NST, bool F16, int EPI, int F, bool ONE, bool HALVES>
__global__ void __launch_bounds__(64 * NWR * NWT, 2) k_prompt_gemm(PromptGemm g) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    bf16x8 *lds = (bf16x8 *)lds_raw;                            // [NST][weight tiles, activation tiles]
    const PromptTile T = prompt_tile(g);
    if constexpr (HALVES) {
        if (T.half >= 0) {
            const int rt0 = (T.rb * WR + T.half * (WR / 2)) * NWR;
            if (rt0 < g.NT) prompt_gemm_tile<WR / 2, WT, NWR, NWT, NST, F16, EPI, F, ONE>(g, rt0, T.tb, T.piece, lds);
            return;
        }
    }
    prompt_gemm_tile<WR, WT, NWR, NWT, NST, F16, EPI, F, ONE>(g, T.rb * WR * NWR, T.tb, T.piece, lds);
}

// ---------------------------------------------------------------------------------------------------
// residual, RMSNorm and operand tiles: one workgroup per token
// ---------------------------------------------------------------------------------------------------
// The pieces of four outputs, added up in order; four requests at a time are on their way.
__device__ __forceinline__ f32x4 sum_pieces(const float *p, size_t step, int n) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int i = 0;
    for (; i + 4 <= n; i += 4) {
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *(const f32x4 *)(p + (size_t)(i + j) * step);
#pragma unroll
        for (int j = 0; j < 4; ++j) s += v[j];
    }
    for (; i < n; ++i) s += *(const f32x4 *)(p + (size_t)i * step);
    return s;
}

constexpr int kRowsMax = 8192;          // inputs (d_model)

// One unit of 8 inputs per thread at d_model 4096 while there are compute units to spare, else two (63 tokens, 8 pieces: 11.1 us with two
// and the pieces requested one after the other, 6.4 now; 1023 tokens, 2 pieces 25 us either way).
template <bool F16, int kRowsThreads>
__global__ void __launch_bounds__(kRowsThreads) k_prompt_rows(PromptRows a) {
    constexpr int kRowsUnits = kRowsMax / 8 / kRowsThreads;     // units per thread
    __shared__ float wsum[kRowsThreads / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    float *x = a.x + (size_t)t * a.d;
    const int nu = a.d / 8;
    f32x4 v[kRowsUnits][2];
    float ssq = 0.f;
#pragma unroll
    for (int i = 0; i < kRowsUnits; ++i) {
        const int u = tid + i * kRowsThreads;
        if (u < nu) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 s = sum_pieces(a.part + (size_t)t * a.d + u * 8 + h * 4, (size_t)a.M * a.d, a.n_split);
                v[i][h] = *(const f32x4 *)(x + u * 8 + h * 4);
                if (a.n_split) {
                    v[i][h] += s;
                    *(f32x4 *)(x + u * 8 + h * 4) = v[i][h];
                }
                ssq += v[i][h][0] * v[i][h][0] + v[i][h][1] * v[i][h][1] + v[i][h][2] * v[i][h][2] + v[i][h][3] * v[i][h][3];
            }
        }
    }
    ssq = sum64(ssq);
    if ((tid & 63) == 0) wsum[tid >> 6] = ssq;
    __syncthreads();
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < kRowsThreads / 64; ++w) total += wsum[w];
    if (tid == 0) a.scale[t] = 1.0f / sqrtf(total * a.inv_dim + a.eps);
#pragma unroll
    for (int i = 0; i < kRowsUnits; ++i) {
        const int u = tid + i * kRowsThreads;
        if (u < nu) {
            float w[8];
            load_w8(a.norm_w, a.elem, (size_t)u * 8, w);
            u16x8 hi, lo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint16_t h, l;
                split16<F16>(v[i][e >> 2][e & 3] * w[e], h, l);
                hi[e] = h;
                lo[e] = l;
            }
            *((u16x8 *)a.B + act_unit(t, u * 8, a.KT, 0)) = hi;
            *((u16x8 *)a.B + act_unit(t, u * 8, a.KT, 1)) = lo;
        }
    }
}

__global__ void __launch_bounds__(256) k_prompt_embed(PromptEmbed a) {
    const int t = a.tok[blockIdx.x];
    for (int c = threadIdx.x * 8; c < a.d; c += 256 * 8) {
        float w[8];
        load_w8(a.table, a.elem, (size_t)t * a.d + c, w);
        float *o = a.out + (size_t)blockIdx.x * a.d + c;
        *(f32x4 *)o = (f32x4){w[0], w[1], w[2], w[3]};
        *(f32x4 *)(o + 4) = (f32x4){w[4], w[5], w[6], w[7]};
    }
}

// ---------------------------------------------------------------------------------------------------
// rotation, KV append, query tiles: one workgroup per 64 (few tokens: 16) tokens and head (q heads, if they are there, then k heads, then v heads)
// ---------------------------------------------------------------------------------------------------
constexpr int kQkvAlign = 64;           // V's dead positions are cleared up to a multiple of this
constexpr int kFewTokens = 256;         // up to here workgroups of 16 tokens, and above of twice the threads per token: larger ones would leave
                                        // compute units idle (63 tokens of the 8B shape: 48 workgroups of 64, 10.6 us, now 192)

template <int DH, int kQkvTokens, bool F16>
__global__ void __launch_bounds__(256) k_prompt_qkv(PromptQkv a) {
    constexpr int half = DH / 2, NC = half / 8;         // groups of 8 dimensions in the lower half
    const int t0 = blockIdx.x * kQkvTokens, head = a.head0 + blockIdx.y, tid = threadIdx.x;
    const int col0 = (int)blockIdx.y * DH;
    auto load8 = [&](int t, int c, float (&o)[8]) {               // columns c .. of this head
        const int col = col0 + c;
        const float *src = a.part + (size_t)t * a.ld + col;
        const size_t step = (size_t)a.M * a.ld;
        const f32x4 s0 = sum_pieces(src, step, a.n_split), s1 = sum_pieces(src + 4, step, a.n_split);
        const float scale = a.scale[t];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = scale * s0[e];
            o[4 + e] = scale * s1[e];
        }
    };
    if (head < a.Hq + a.Hkv) {
        const bool is_q = head < a.Hq;
        for (int idx = tid; idx < kQkvTokens * NC; idx += 256) {
            const int tl = idx / NC, c = idx % NC, t = t0 + tl;
            if (t >= a.M) break;
            float x[8], y[8], r0[8], r1[8];
            load8(t, c * 8, x);
            load8(t, half + c * 8, y);
            const float *rp = a.rope + ((size_t)t * half + c * 8) * 2;
            const float mul = is_q ? a.q_scale : 1.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float cs = rp[2 * e], sn = rp[2 * e + 1];
                r0[e] = x[e] * cs - y[e] * sn;
                r1[e] = x[e] * sn + y[e] * cs;
                if (is_q) {
                    r0[e] *= mul;
                    r1[e] *= mul;
                }
            }
            if (is_q) {
                // query row t * G + (head in group) of its kv head; tiles of 16 rows over DH inputs
                const int kvh = head / a.G, r = t * a.G + (head - kvh * a.G);
                u16x8 *Q = (u16x8 *)a.Q + (size_t)kvh * (size_t)(a.q_rows / 16) * (DH / 32) * 128;
                u16x8 h0, l0, h1, l1;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    uint16_t hi, lo;
                    split16<F16>(r0[e], hi, lo);
                    h0[e] = hi;
                    l0[e] = lo;
                    split16<F16>(r1[e], hi, lo);
                    h1[e] = hi;
                    l1[e] = lo;
                }
                Q[act_unit(r, c * 8, DH / 32, 0)] = h0;
                Q[act_unit(r, c * 8, DH / 32, 1)] = l0;
                Q[act_unit(r, half + c * 8, DH / 32, 0)] = h1;
                Q[act_unit(r, half + c * 8, DH / 32, 1)] = l1;
            } else {
                uint16_t *K = (uint16_t *)a.Kc + ((size_t)(head - a.Hq) * a.stride + a.pos0 + t) * DH;
                u16x8 k0, k1;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    k0[e] = to16<F16>(r0[e]);
                    k1[e] = to16<F16>(r1[e]);
                }
                *(u16x8 *)(K + c * 8) = k0;
                *(u16x8 *)(K + half + c * 8) = k1;
            }
        }
    } else {
        // V is kept transposed: through LDS, then 8 positions of a dimension per store.  Positions past the prompt, up to the
        // next multiple of 64 (within the cache row), are dead; they get zeros, which the attention kernel may multiply by 0.
        __shared__ uint16_t vt[DH][kQkvTokens + 8];
        const int h = head - a.Hq - a.Hkv;
        for (int idx = tid; idx < kQkvTokens * (DH / 8); idx += 256) {
            const int tl = idx / (DH / 8), c = idx % (DH / 8), t = t0 + tl;
            float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (t < a.M) load8(t, c * 8, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) vt[c * 8 + e][tl] = to16<F16>(x[e]);
        }
        __syncthreads();
        uint16_t *V = (uint16_t *)a.Vc + (size_t)h * DH * a.stride + a.pos0 + t0;
        for (int idx = tid; idx < DH * (kQkvTokens / 8); idx += 256) {
            const int e = idx / (kQkvTokens / 8), p = idx % (kQkvTokens / 8);
            *(u16x8 *)(V + (size_t)e * a.stride + p * 8) = *(const u16x8 *)&vt[e][p * 8];
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// attention: one workgroup per kv head and 64 query rows (row r = token r / G, head r % G of the group)
// ---------------------------------------------------------------------------------------------------
// The products are those of the decode kernel (ad_attention_device.h): S^T = K q^T with the rows of the two score tiles
// assigned to keys so that a lane ends up with 8 consecutive keys of its query row, which is the B operand layout of
// O^T = V^T P^T; queries and probabilities are split hi/lo.  A wavefront holds 16 query rows; the workgroup's four
// wavefronts share the K and V tiles of 64 positions, copied into LDS one block ahead without a way through registers, and run the softmax
// online.  Bound by the chain through a block (scores, softmax, second product) more than by its arithmetic: 16 rows a wavefront and twice
// the workgroups beat 32 (1024 tokens of the 8B shape 45.1 against 55.7 us), and blocks of 64 positions, whose two halves go through the chain side by
// side, beat 32: 8B shape, 299 / 511 / 1023 tokens 15.3 / 23.2 / 48.2 -> 14.3 / 20.1 / 40.6 us, 13B 16.5 (299) / 47.3 (1023) -> 14.4 / 41.6.
constexpr int kPromptAttnRows = 64;

template <int DH, bool F16>
__global__ void __launch_bounds__(256, 2) k_prompt_attn(PromptAttn a) {
    constexpr int KS = DH / 32, DT = DH / 16;
    constexpr int KU = 2 * KS * 64, VU = DT * 64, HU = KU + VU;  // 16-byte units of 32 positions: K tiles, V tiles, both
    constexpr int NC = 2 * HU / 64 / 4;                          // copies of 1 KiB per wavefront and block
    __shared__ bf16x8 lds[2][2 * HU];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, gq = lane >> 4;
    const int kvh = blockIdx.x % a.Hkv, n_blk = (a.M * a.G + kPromptAttnRows - 1) / kPromptAttnRows;
    const int blk = n_blk - 1 - blockIdx.x / a.Hkv;              // the blocks with the most keys first
    const int R = a.M * a.G, r_blk = blk * kPromptAttnRows;
    const int r_last = (r_blk + kPromptAttnRows < R ? r_blk + kPromptAttnRows : R) - 1;
    const int n_key = a.pos0 + r_last / a.G + 1;                 // keys the block's last row sees
    const int n_kb = (n_key + 63) / 64;

    const uint16_t *Kg = (const uint16_t *)a.Kc + (size_t)kvh * a.stride * DH;
    const uint16_t *Vg = (const uint16_t *)a.Vc + (size_t)kvh * DH * a.stride;
    // A block of 64 positions in LDS: of each half its K tiles [aa][j][lane], then its V tiles [dt][lane].  A block lies inside the cache row
    // (stride and pos0 are multiples of 64); positions at or past the row's end of keys are masked.
    unsigned src[NC];                                            // byte offset of this lane's 16 bytes in the first block
    bool is_k[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int t = wave * NC + i, h = t / (HU / 64), u = t % (HU / 64);      // half, tile of it
        is_k[i] = u < 2 * KS;
        if (is_k[i]) src[i] = ((unsigned)(h * 32 + 8 * (n >> 2) + 4 * (u / KS) + (n & 3)) * DH + (u % KS) * 32 + gq * 8) * 2u;
        else src[i] = ((unsigned)((u - 2 * KS) * 16 + n) * (unsigned)a.stride + h * 32 + gq * 8) * 2u;
    }
    auto copy = [&](int kb, int buf) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const char *base = is_k[i] ? (const char *)Kg + (size_t)kb * 64 * DH * 2 : (const char *)Vg + (size_t)kb * 128;
            copy_to_lds(base + src[i], &lds[buf][(wave * NC + i) * 64]);
        }
    };
    copy(0, 0);

    const int row0 = r_blk + wave * 16, row = row0 + n;          // this wavefront's first row, this lane's row
    const bf16x8 *Q = (const bf16x8 *)a.Q + ((size_t)kvh * (a.q_rows / 16) + row0 / 16) * KS * 128;
    const int t_row = (row < R ? row : R - 1) / a.G, see = a.pos0 + t_row;      // its token and last visible position
    bf16x8 q[KS][2];
#pragma unroll
    for (int j = 0; j < KS; ++j)
#pragma unroll
        for (int p = 0; p < 2; ++p) q[j][p] = Q[(j * 2 + p) * 64 + lane];
    const int w_last = (row0 + 16 < R ? row0 + 16 : R) - 1;
    const int w_key = row0 < R ? a.pos0 + w_last / a.G + 1 : 0;  // keys this wavefront's last row sees
    const int w_full = row0 < R ? a.pos0 + row0 / a.G + 1 : 0;   // keys all its rows see

    constexpr float kPScale = F16 ? 1024.0f : 1.0f;              // keeps small probabilities out of fp16's subnormals
    f32x4 o[DT];
    float mx = -INFINITY, sum = 0.f;
#pragma unroll
    for (int d = 0; d < DT; ++d) o[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int kb = 0; kb < n_kb; ++kb) {
        // this block's copies have landed, everyone's, and nobody reads the other buffer any more
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (kb + 1 < n_kb) copy(kb + 1, (kb + 1) & 1);
        const bf16x8 *cur = lds[kb & 1];
        if (kb * 64 < w_key) {
            f32x4 s[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) s[h][0] = s[h][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < KS; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int aa = 0; aa < 2; ++aa) s[h][aa] = mma16<F16>(cur[h * HU + (aa * KS + j) * 64 + lane], q[j][p], s[h][aa]);
            const bool masked = kb * 64 + 64 > w_full;           // some row of this wavefront does not see the whole block
            float sc[16], bm = -INFINITY;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                sc[c] = s[c >> 3][(c >> 2) & 1][c & 3];
                if (masked && kb * 64 + (c >> 3) * 32 + gq * 8 + (c & 7) > see) sc[c] = -INFINITY;
                bm = fmaxf(bm, sc[c]);
            }
            bm = max_rows(bm);
            const float nm = fmaxf(mx, bm), ref = softmax_ref(nm);
            const float alpha = __expf(mx - ref);
            mx = nm;
            float add = 0.f;
            u16x8 h8[2], l8[2];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const float p = __expf(sc[c] - ref);
                add += p;
                uint16_t hi, lo;
                split16<F16>(p * kPScale, hi, lo);
                h8[c >> 3][c & 7] = hi;
                l8[c >> 3][c & 7] = lo;
            }
            sum = sum * alpha + add;
            if (!__all(alpha == 1.0f)) {
#pragma unroll
                for (int d = 0; d < DT; ++d) o[d] *= alpha;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h && kb * 64 + 32 >= w_key) break;           // (none of its rows sees a key there: no weights of 0 for entries that may be infinite)
                const bf16x8 ph = __builtin_bit_cast(bf16x8, h8[h]), pl = __builtin_bit_cast(bf16x8, l8[h]);
#pragma unroll
                for (int d = 0; d < DT; ++d) o[d] = mma16<F16>(cur[h * HU + KU + d * 64 + lane], ph, o[d]);
#pragma unroll
                for (int d = 0; d < DT; ++d) o[d] = mma16<F16>(cur[h * HU + KU + d * 64 + lane], pl, o[d]);
            }
        }
    }
    // lane (n, gq): query row n of the tile, dims d*16 + gq*4 .. +3
    sum = sum_rows(sum);
    const float inv = 1.0f / (sum * kPScale);
    if (row < R) {
        const int hq = kvh * a.G + (row - t_row * a.G);
#pragma unroll
        for (int d = 0; d < DT; ++d) {
            u16x4 h4, l4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint16_t hi, lo;
                split16<F16>(o[d][e] * inv, hi, lo);
                h4[e] = hi;
                l4[e] = lo;
            }
            const int k = hq * DH + d * 16 + (gq >> 1) * 8;
            *(u16x4 *)((uint16_t *)((bf16x8 *)a.Bo + act_unit(t_row, k, a.Bo_KT, 0)) + (gq & 1) * 4) = h4;
            *(u16x4 *)((uint16_t *)((bf16x8 *)a.Bo + act_unit(t_row, k, a.Bo_KT, 1)) + (gq & 1) * 4) = l4;
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------
template <int WR, int WT, int NWR, int NWT, int NST, bool ONE, bool F16, int EPI, int F>
int launch_gemm_flush(const PromptGemm &g, hipStream_t s) {
    constexpr bool HALVES = WR == 4;
    constexpr int lds = NST * prompt_stage_units(WR * NWR, WT * NWT) * 16;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_prompt_gemm<WR, WT, NWR, NWT, NST, F16, EPI, F, ONE, HALVES>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    const int tiles = g.n_rb * g.n_tb * g.n_split, grid = g.n_full + 2 * (tiles - g.n_full);
    hipLaunchKernelGGL((k_prompt_gemm<WR, WT, NWR, NWT, NST, F16, EPI, F, ONE, HALVES>), dim3(grid), dim3(64 * NWR * NWT), lds, s, g);
    return (int)hipGetLastError();
}
template <int WR, int WT, int NWR, int NWT, int NST, bool ONE, bool F16, int EPI>
int launch_gemm_as(const PromptGemm &g, hipStream_t s) {
    if (g.k_per > kLongPiece) return launch_gemm_flush<WR, WT, NWR, NWT, NST, ONE, F16, EPI, kFlushLong>(g, s);
    return launch_gemm_flush<WR, WT, NWR, NWT, NST, ONE, F16, EPI, kFlush>(g, s);
}

template <bool F16, int EPI>
int launch_gemm_sized(PromptGemm g, int n_wg, int *n_split, hipStream_t s) {
    if (EPI == PG_PART && (size_t)g.M * g.N > g.part_floats) return (int)hipErrorInvalidValue;
    const int kind = choose_prompt_tile(g, EPI == PG_PART, n_wg);
    if (n_split) *n_split = g.n_split;
    switch (kind) {
        case 0: return launch_gemm_as<1, 2, 4, 1, 8, true, F16, EPI>(g, s);
        case 1: return launch_gemm_as<2, 2, 4, 1, 5, true, F16, EPI>(g, s);
        case 2: return launch_gemm_as<2, 2, 4, 2, 5, true, F16, EPI>(g, s);
        case 3: return launch_gemm_as<2, 3, 4, 2, 4, false, F16, EPI>(g, s);
        case 4: return launch_gemm_as<2, 4, 4, 2, 4, false, F16, EPI>(g, s);
        case 5: return launch_gemm_as<3, 3, 4, 2, 4, false, F16, EPI>(g, s);
        case 6: return launch_gemm_as<3, 4, 4, 2, 4, false, F16, EPI>(g, s);
        case 7: return launch_gemm_as<4, 3, 4, 2, 4, false, F16, EPI>(g, s);
        default: return launch_gemm_as<4, 4, 4, 2, 4, false, F16, EPI>(g, s);
    }
}

}  // namespace

int launch_prompt_gemm(PromptGemm g, bool swiglu, int n_wg, int *n_split, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    if (g.M < 1 || g.M > kPromptRows || g.NT < 1 || g.KT < 1) return (int)hipErrorInvalidValue;
    if (swiglu) return g.f16 ? launch_gemm_sized<true, PG_SWIGLU>(g, n_wg, n_split, s) : launch_gemm_sized<false, PG_SWIGLU>(g, n_wg, n_split, s);
    return g.f16 ? launch_gemm_sized<true, PG_PART>(g, n_wg, n_split, s) : launch_gemm_sized<false, PG_PART>(g, n_wg, n_split, s);
}

int launch_prompt_embed(const PromptEmbed &a, void *stream) {
    if (a.n < 1 || a.n > kPromptEmbedRows) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prompt_embed, dim3(a.n), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_prompt_rows(const PromptRows &a, void *stream) {
    if (a.M < 1 || a.d > kRowsMax || a.elem == kElemF32) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    const bool f16 = a.elem == kElemF16;
    if (a.M <= kFewTokens) {
        if (f16) hipLaunchKernelGGL((k_prompt_rows<true, 512>), dim3(a.M), dim3(512), 0, s, a);
        else hipLaunchKernelGGL((k_prompt_rows<false, 512>), dim3(a.M), dim3(512), 0, s, a);
    } else {
        if (f16) hipLaunchKernelGGL((k_prompt_rows<true, 256>), dim3(a.M), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_prompt_rows<false, 256>), dim3(a.M), dim3(256), 0, s, a);
    }
    return (int)hipGetLastError();
}

template <int DH, bool F16>
static int launch_qkv_as(const PromptQkv &a, hipStream_t s) {
    const int n = (a.M + kQkvAlign - 1) / kQkvAlign * kQkvAlign, heads = a.Hq + 2 * a.Hkv - a.head0;
    if (a.M <= kFewTokens) hipLaunchKernelGGL((k_prompt_qkv<DH, 16, F16>), dim3(n / 16, heads), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_prompt_qkv<DH, 64, F16>), dim3(n / 64, heads), dim3(256), 0, s, a);
    return (int)hipGetLastError();
}
int launch_prompt_qkv(const PromptQkv &a, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    if (a.pos0 % kQkvAlign) return (int)hipErrorInvalidValue;
    if (a.dh == 128) return a.f16 ? launch_qkv_as<128, true>(a, s) : launch_qkv_as<128, false>(a, s);
    if (a.dh == 64) return a.f16 ? launch_qkv_as<64, true>(a, s) : launch_qkv_as<64, false>(a, s);
    return (int)hipErrorInvalidValue;
}

template <int DH, bool F16>
static int launch_attn_as(const PromptAttn &a, hipStream_t s) {
    const int n_blk = (a.M * a.G + kPromptAttnRows - 1) / kPromptAttnRows;
    hipLaunchKernelGGL((k_prompt_attn<DH, F16>), dim3(n_blk * a.Hkv), dim3(256), 0, s, a);
    return (int)hipGetLastError();
}
int launch_prompt_attn(const PromptAttn &a, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    if (a.dh == 128) return a.f16 ? launch_attn_as<128, true>(a, s) : launch_attn_as<128, false>(a, s);
    if (a.dh == 64) return a.f16 ? launch_attn_as<64, true>(a, s) : launch_attn_as<64, false>(a, s);
    return (int)hipErrorInvalidValue;
}

}  // namespace ad
