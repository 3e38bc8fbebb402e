// Prints the host plan of linear layers (linear_plan.cpp), one line per layer
// read from stdin: k, 16 moduli, batch, c_in, h_in, w_in, c_out, kh, kw,
// stride, pad.  A refused layer prints its return code alone.
#include <stdio.h>
#include <string.h>

#include "../paper_2506_14489_amd/csrc/linear_plan.hpp"

using namespace redash;

int main() {
    uint32_t v[26];
    for (;;) {
        for (uint32_t &x : v)
            if (scanf("%u", &x) != 1) return 0;
        redash_linear_params p;
        memset(&p, 0, sizeof p);
        p.k = v[0];
        memcpy(p.moduli, v + 1, sizeof p.moduli);
        p.batch = v[17], p.c_in = v[18], p.h_in = v[19], p.w_in = v[20], p.c_out = v[21];
        p.kh = v[22], p.kw = v[23], p.stride = v[24], p.pad = v[25];
        LinPlan L;
        const int rc = build_lin_plan(&p, &L);
        if (rc) {
            printf("rc=%d\n", rc);
            continue;
        }
        printf("rc=0 ncc=%u ck=%u kh=%u kw=%u flat=%u xt=%u word_split=%u og_xcd=%u fold_c=%u wp=%u xlast=%u cp=%u "
               "xtiles=%u tile_rows=%u lds_bytes=%u plane_bytes=%llu\n",
               L.ncc, L.ck, L.kh, L.kw, L.flat, L.xt, L.word_split, L.og_xcd, L.fold_c, L.wp, L.xlast, L.cp, L.xtiles,
               L.tile_rows, L.lds_bytes, static_cast<unsigned long long>(L.plane_bytes));
    }
}
