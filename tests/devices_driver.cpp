// Calls of the library on streams of two devices, with either of them current, against stand-ins for the runtime: a kernel's handle has to be
// one of the stream's device.  (Launches by the host function's address leave the choice to the runtime.)  Nothing runs on a GPU.
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "adadecode.h"

static int current = 0, wrong = 0, by_handle = 0, by_address = 0;
struct Stream { int device; };
static Stream streams[2] = {{0}, {1}};
static int device_of(hipStream_t s) { return s && s != hipStreamLegacy && s != hipStreamPerThread ? ((Stream *)s)->device : current; }

extern "C" {
hipError_t hipGetDevice(int *d) { *d = current; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) {
    if (s == hipStreamLegacy || s == hipStreamPerThread) abort();       // (the runtime takes the former for an address)
    *d = device_of(s);
    return hipSuccess;
}
hipError_t hipGetFuncBySymbol(hipFunction_t *f, const void *symbol) {
    *f = (hipFunction_t)((uintptr_t)symbol << 1 | (unsigned)current);
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, hipStream_t s, void **, void **) {
    ++by_handle;
    if ((int)((uintptr_t)f & 1) != device_of(s)) ++wrong;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { ++by_address; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char word[256]; *p = word; return hipSuccess; }
}

#define OK(x) do { if ((x) != AD_OK) { printf("%s: %s\n", #x, ad_last_error()); return 1; } } while (0)

static int calls(const ad_model *m, ad_kv *kv, char *mem, void *stream) {
    const int32_t tok[3] = {1, 2, 3}, pos[3] = {700, 701, 702}, draft[2] = {1, 2};
    const float u[2] = {0.5f, 0.5f};
    int32_t *out = (int32_t *)mem;
    for (int l = 1; l <= 2; ++l) OK(ad_kv_set_len(kv, l, 700));
    OK(ad_embed(m, tok, 3, mem, stream));
    OK(ad_layer_steps(m, kv, 1, 2, mem, pos, 3, stream));
    OK(ad_exit_head(m, 1, mem, out, (float *)out + 1, stream));
    OK(ad_verify(m, mem, draft, 3, out, out + 1, out + 2, stream));
    OK(ad_head_logits(m, 2, mem, 3, mem, stream));
    OK(ad_sample_logits(m, mem, 0.8f, 0.5f, out, (float *)out + 1, stream));
    OK(ad_verify_sampled(m, mem, mem, draft, 3, 0.8f, u, u, 0.5f, out, out + 1, (float *)out + 2, stream));
    return 0;
}

int main() {
    for (int dtype : {AD_BF16, AD_F32}) {
        ad_config c;
        memset(&c, 0, sizeof c);
        c.n_layers = 2; c.d_model = 256; c.n_q_heads = 4; c.n_kv_heads = 2; c.head_dim = 64; c.d_ffn = 512; c.vocab = 9000; c.dtype = dtype;
        c.rope_base = 10000.f; c.rms_eps = 1e-5f; c.m_max = 8; c.n_exit = 1; c.exit_layers[0] = 1;
        const size_t ws = ad_workspace_bytes(&c), kb = ad_kv_bytes(&c, 1000);
        std::vector<char> mem(1 << 20);
        char *w = (char *)aligned_alloc(256, (ws + 255) / 256 * 256), *k = (char *)aligned_alloc(256, (kb + 255) / 256 * 256), *p = mem.data();
        ad_layer_weights lw[2];
        for (auto &l : lw) l.attn_norm = l.wq = l.wk = l.wv = l.wo = l.ffn_norm = l.w_gate = l.w_up = l.w_down = p;
        ad_top_weights top;
        memset(&top, 0, sizeof top);
        top.embed = top.final_norm = top.lm_head = p;
        ad_model *m = nullptr;
        ad_kv *kv = nullptr;
        current = 1;
        OK(ad_model_create(&c, lw, &top, w, ws, &streams[1], &m));
        OK(ad_kv_create(m, k, kb, 1000, &streams[1], &kv));
        // the model's device is 1; the first calls come from a thread with device 0 current, the others with either
        const struct { int current; void *stream; } turns[] = {{0, &streams[1]}, {1, &streams[1]}, {0, &streams[1]}, {1, nullptr}, {0, nullptr}, {0, &streams[0]}, {1, &streams[0]},
                                                          {1, hipStreamLegacy}, {0, hipStreamPerThread}};
        for (const auto &t : turns) {
            current = t.current;
            wrong = by_handle = by_address = 0;
            if (calls(m, kv, p, t.stream)) return 1;
            printf("dtype %d, device %d current, stream of %d: %d launches by handle, %d by address, %d of another device\n", dtype, current,
                   device_of((hipStream_t)t.stream), by_handle, by_address, wrong);
            if (wrong || by_handle + by_address != 21 || ((t.stream == hipStreamLegacy || t.stream == hipStreamPerThread) && by_handle)) return 1;
        }
        ad_kv_destroy(kv);
        ad_model_destroy(m);
        free(w);
        free(k);
    }
    printf("every launch on its stream's device\n");
    return 0;
}
