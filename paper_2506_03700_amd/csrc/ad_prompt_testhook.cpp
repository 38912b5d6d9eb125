// CPU-only test hook: how the prompt pass lays a projection out.  Built into libad_sched_test.so, never into the product library.
#include <string.h>

#include "ad_prompt_layout.h"

// out: kind of tile, pieces along K, k-steps per piece, workgroups, whole tiles among them, fewest pieces
extern "C" void ad_prompt_test_layout(int N, int K, int M, size_t part_floats, int swiglu, int n_wg, int *out) {
    ad::PromptGemm g;
    memset(&g, 0, sizeof g);
    g.NT = N / 16; g.KT = (K + 31) / 32; g.N = N; g.M = M; g.part_floats = part_floats;
    out[0] = ad::choose_prompt_tile(g, !swiglu, n_wg);
    out[1] = g.n_split;
    out[2] = g.k_per;
    out[3] = g.n_full + 2 * (g.n_rb * g.n_tb * g.n_split - g.n_full);
    out[4] = g.n_full;
    out[5] = swiglu ? 1 : ad::fewest_pieces(g, n_wg);
}
