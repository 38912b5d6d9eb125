// Calls the launchers of the projections' kernels with arguments that these kernels have no form for: each has to be refused before
// anything is launched (hipErrorInvalidValue), with a GPU or without one.
#include <stdio.h>
#include <string.h>

#include "ad_internal.h"

using namespace ad;

static int failures = 0;
static void refused(const char *what, int rc) {
    printf("%-60s %d\n", what, rc);
    if (rc != 1) ++failures;
}

int main() {
    static float x[8 * 4096], w[4096], out[8 * 4096];
    const LaunchCtx ctx{nullptr, 256};
    const struct { int elem, planes; const char *name; } types[] = {{kElemF32, 3, "fp32"}, {kElemBF16, 1, "bf16"}, {kElemF16, 1, "fp16"}};
    for (const auto &t : types) {
        GemmArgs g;
        memset(&g, 0, sizeof g);
        g.elem = t.elem; g.NT = 4; g.KT = 2; g.N = 64; g.K = 64; g.m = 1; g.ld = 64; g.out = out; g.resid = x;
        g.mode = GEMM_STATIONARY;
        g.epi = EPI_RESID;
        printf("%s\n", t.name);
        g.W = w; g.B = w;
        refused("many row tiles: a residual", launch_rows(g, t.planes, 4, ctx));
        g.B = nullptr; g.x = x; g.ldx = 64; g.norm_w = w;
        refused("many row tiles: fp32 rows and a residual", launch_rows(g, t.planes, 4, ctx));
        refused("few row tiles: fp32 rows and a residual", launch_proj(g, t.planes, ctx));
        g.epi = EPI_STORE; g.norm_w = nullptr;
        refused("many row tiles: fp32 rows without norm weights", launch_rows(g, t.planes, 4, ctx));
        refused("few row tiles: fp32 rows without norm weights", launch_proj(g, t.planes, ctx));
        g.norm_w = w; g.K = 4096 + 32; g.KT = g.K / 32;
        refused("few row tiles: more inputs than two batches a wavefront", launch_proj(g, t.planes, ctx));
    }
    printf(failures ? "FAILED\n" : "all refused\n");
    return failures != 0;
}
