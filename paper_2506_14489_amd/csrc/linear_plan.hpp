// Host-side plan of a garbled linear layer: validation, the tiles, the LDS
// layout, the residue planes and the launch shape of the layer kernels
// (linear.hip), which receive it by value.
#pragma once

#include <stdint.h>

#include "../../include/redash.h"
#include "plan.hpp"

namespace redash {

constexpr int kLinBlock = 256;      // 4 waves
constexpr int kLinOTile = 64;       // output channels per workgroup
constexpr uint32_t kLinMaxLds = 160 * 1024;
constexpr uint32_t kLinMaxK = 16384;  // c_in kh kw (the epilogue bounds below)
constexpr uint32_t kLinMaxTaps = 64;
constexpr uint32_t kLinMaxPairs = 96;  // (modulus, packed word) pairs: sum of W <= 15 * 6
constexpr int kXcds = 8;               // MI355X: workgroups go round-robin to 8 XCDs

struct LinMod {
    uint32_t m, b, g, W, glast;
    uint32_t woff;     // word offset of this modulus's block (in units of n)
    // Residue planes: a plane byte holds f = 8 / bp residues of bp bits
    // (m <= 16: m = 2 eight of one bit, 3 and 4 four of two bits, 5..16 two
    // of four bits) or one residue byte (m > 16).  Plane pn(w, j) = w ppw +
    // j / f of this modulus holds field j mod f of residues j of packed word w.
    uint32_t pl_off;   // planes of the earlier moduli
    uint32_t bp, lgf;  // bits per field in a plane byte, log2 f
    uint32_t ppw;      // planes per full packed word: ceil(g / f)
    uint32_t rep;      // a bp-bit mask in every byte (f > 1)
    // floor(u / m) = umulhi(u, divM) >> divS for every u the epilogue sees
    uint32_t divM, divS;
    uint32_t off;      // a multiple of m above |sum w v|: keeps u >= 0
};

struct LinPlan {
    uint32_t k;
    uint32_t c_in, c_out, kh, kw, stride, pad;
    uint32_t in_rows, in_cols;    // input rows and columns of one image (dense: 1, batch)
    uint32_t rows, cols, nimg;    // output rows, columns, images (dense: 1, batch, 1)
    uint32_t sN, sC, sY, sX;      // input activation index = img sN + c sC + y sY + x sX
    uint32_t oN, oO, oY, oX;      // output activation index, likewise
    uint32_t hp, wp, cp;          // plane rows and columns (padded) and channel bytes per position
                                  // (ncc ck; folded: the layer's own c_in)
    uint32_t xt, xtiles;          // output positions per tile, tiles per row
    uint32_t ck, kc, taps, ncc;   // channel chunk, K bytes per chunk (64-padded), kh kw, chunks
    uint32_t lg_ck;
    uint32_t kw_magic;            // floor(t / kw) = (t kw_magic) >> 16 for every tap t < 64
    uint32_t o_pad, ogroups;      // c_out rounded up to 64, its groups of 64
    uint32_t astride;             // LDS bytes per staged weight row
    uint32_t ostride;             // words per output-channel row of the merged output words
    uint32_t xw, xstride;         // staged input columns of a tile; LDS bytes per staged column
    uint32_t gstep, lstep;        // plane columns between staged ones; staged columns between outputs
    uint32_t xlast;               // the last plane column that is staged
    uint32_t wpair;               // staging: the two columns of an 8-lane write group lie wpair apart
    uint32_t halo;                // LDS bytes of one residue's staged input (kh xw xstride)
    uint32_t lds_a, lds_b, lds_o, lds_bytes;
    uint32_t npairs;
    uint32_t word_split;          // k_linear_gemm: one workgroup per packed word (else per modulus)
    uint32_t og_xcd;              // k_linear_gemm: output channel groups dealt to the XCDs (see the plan)
    uint32_t fold_c;              // column fold (see the plan): the layer's own c_in, else 0
    uint32_t flat, tile_rows;     // k_linear_gemm over the flattened plane (see the plan); rows of tiles
    uint64_t n_in, n_out;         // activations
    uint64_t plane_bytes;         // nimg hp wp cp
    uint64_t rowsum_off;          // byte offset of the row sums in the prepared buffer
    uint32_t total_planes;        // residue planes over the base
    uint8_t pair_mod[kLinMaxPairs], pair_word[kLinMaxPairs];
    LinMod mod[kMaxK];
};

// Builds and validates the plan.  Returns REDASH_OK, REDASH_E_NULL or
// REDASH_E_PARAM.
int build_lin_plan(const redash_linear_params *p, LinPlan *out);

// Buffer sizes of a plan: prepared weights, working buffer (bytes), and the
// label words per activation.
uint64_t prepared_bytes(const LinPlan &L);
uint64_t work_bytes(const LinPlan &L);
uint32_t total_words(const LinPlan &L);

}  // namespace redash
