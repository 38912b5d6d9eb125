// The prompt pass ("KV cache <- LM(x)" of Algorithm 1): argument blocks and launchers of ad_prompt.hip, which runs up
// to kPromptRows prompt tokens through a layer at once.  16-bit models only.  Not installed.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace ad {

// ---- operand layout ------------------------------------------------------------------------------------
// Activations [M tokens, K] -> tiles of 16 tokens x 32 inputs in two planes, the 16-bit hi and lo parts (x = hi + lo):
// tile (tt, ks) is 2 KiB, [plane][lane][8 inputs], lane l holding token tt*16 + (l & 15) and inputs
// ks*32 + (l >> 4)*8 .. +8: the B operand of one 16x16x32 MFMA, as the weight tiles (ad_internal.h) are its A operand.
// Tiles are ordered [tt][ks].
constexpr int kPromptAlign = 128;     // tokens of the largest workgroup tile
constexpr int kPromptRows = 1024;     // most tokens per pass through the layers (a multiple of kPromptAlign)
// Fewest tokens it is used for; up to 8 are one layer step per layer.  A whole ad_generate of one token, prompt pass against layer
// steps, 9 / 16 / 33 tokens before the last: 8B shape, 8 layers 1.50 / 1.51 / 1.61 against 2.13 / 2.25 / 4.45 ms, tiny bf16 model
// 0.22 / 0.22 / 0.23 against 0.28 / 0.29 / 0.54 ms; for 8 tokens one layer step per layer takes 1.47 ms (8B).
constexpr int kPromptMin = 9;
constexpr int kPromptMaxSplit = 8;    // most pieces a contraction is cut into along K

inline size_t prompt_act_bytes(int64_t rows, int64_t K) { return (size_t)rows * (size_t)((K + 31) / 32 * 32) * 4u; }
// floats of the partial products of the projections that store fp32 rows (one [M][N] block per piece of K): whole for
// the widest, at least two pieces for the projections onto d
inline size_t prompt_part_floats(int64_t rows, int64_t nqkv, int64_t d) { return (size_t)rows * (size_t)(nqkv > 2 * d ? nqkv : 2 * d); }

// out[t][n] = sum_k W[n][k] act[t][k]
struct PromptGemm {
    const void *W, *B;        // packed weights (one plane), activation tiles
    int NT, KT, N, M;         // row tiles, k-steps, valid output rows, tokens
    float *part;              // [pieces][M][N] fp32 (swiglu: unused)
    size_t part_floats;       // room there
    const float *scale;       // swiglu: 1 / rms of each token's input row
    void *Bnext;              // swiglu: activation tiles of the next projection, Bnext_KT k-steps
    int Bnext_KT;
    int f16;                  // fp16 operands (else bf16)
    // set by the launcher: tiles along the rows and along the tokens, pieces along K and k-steps per piece; tiles that are a workgroup each
    // (the rest are two)
    int n_rb, n_tb, n_split, k_per, n_full;
};

// x[t] (+)= sum of the pieces; activation tiles of x[t] * w, and the factor 1 / rms(x[t]) that makes RMSNorm of it, which
// the projection's consumer applies (the embedding rows and norm weights of a 16-bit model have products that the split
// keeps exactly; multiplied by the factor first, they lose that)
struct PromptRows {
    float *x;                 // [M][d], updated in place if there are pieces
    const float *part;        // [n_split][M][d]
    int n_split, M, d, KT;
    const void *norm_w;       // 16-bit, elem
    int elem;
    float inv_dim, eps;
    void *B;
    float *scale;             // [M]
};

// q, k, v of M tokens from the pieces: rotated and scaled queries in operand tiles, K and V into the cache
struct PromptQkv {
    const float *part;        // [n_split][M][ld]: heads head0 .. of q, k, v
    const float *scale;       // [M], see PromptRows
    int n_split, M, ld, head0, Hq, Hkv, dh, G;
    const float *rope;        // rows pos0 ..
    void *Kc, *Vc;            // the layer's cache (see AttnArgs)
    int stride, pos0;         // pos0: a multiple of 64
    int q_rows;               // query rows of a kv head that Q has room for
    void *Q;                  // per kv head, query rows r = t * G + head in group: tiles of 16 rows, [tile][ks][plane][lane][8]
    float q_scale;            // 1 / sqrt(dh)
    int f16;
};

struct PromptAttn {
    const void *Q, *Kc, *Vc;
    int stride, pos0, M, Hq, Hkv, dh, G, q_rows;
    void *Bo;                 // activation tiles of the Wo projection
    int Bo_KT, f16;
};

constexpr int kPromptEmbedRows = 512;      // token ids travel in the kernel arguments
struct PromptEmbed { const void *table; int elem, d, n; float *out; int32_t tok[kPromptEmbedRows]; };

int launch_prompt_embed(const PromptEmbed &, void *stream);
int launch_prompt_rows(const PromptRows &, void *stream);
// n_wg: compute units.  *n_split: pieces the product was cut into (null for swiglu, which is never cut).
int launch_prompt_gemm(PromptGemm g, bool swiglu, int n_wg, int *n_split, void *stream);
int launch_prompt_qkv(const PromptQkv &, void *stream);
int launch_prompt_attn(const PromptAttn &, void *stream);

}  // namespace ad
