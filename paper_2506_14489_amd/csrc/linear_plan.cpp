// Host-side plan of a garbled linear layer.
#include "linear_plan.hpp"

#include <string.h>

namespace redash {

namespace {

uint32_t gcd32(uint32_t a, uint32_t b) {
    while (b) {
        const uint32_t r = a % b;
        a = b;
        b = r;
    }
    return a;
}

uint32_t round_up(uint32_t v, uint32_t q) { return (v + q - 1) / q * q; }

// The forms of a 3x3 stride-1 layer over several 64-channel chunks: 16-position
// tiles of a row, or 16- or 32-position tiles of the flattened plane, each with
// a workgroup per modulus or per packed word.
//
// Estimated time of one (us, up to a part that is the same for all): a stage
// (four residues of a word, one chunk) on each of the 512 workgroups that run
// together costs `stage` and `column` for each 100 staged columns, a workgroup
// `start`, the stages of the longest workgroup `serial` each (the launch ends
// with such a one), the launch `fixed`.  Fitted to the times of 700 layers (65 to
// 512 channels, 16 to 512 outputs, 4 to 36 columns, batch 1 to 16, four bases;
// relative error 6-11%).  Over them the form chosen is on geometric mean 0.6%
// slower than the fastest of the six, and over 150 others 15% faster than row
// tiles for more than 8 columns and 7% faster than flattened tiles everywhere,
// which cost rows of 16 or 32 positions and small or unevenly filled grids up to
// 40% (128 -> 128 channels at 16x16 71 us in rows, 82 flattened; 8 primes, 192 ->
// 64 at 32x32 138 and 191; 512 -> 512 at 8x8, batch 8, 2.07 ms at 16 positions,
// 2.81 at 32, 1.78 at 16 with a workgroup per word).
struct FormCost {
    double stage, column, serial, start, fixed;
};
constexpr FormCost kFormCost[3][2] = {
    // {a workgroup per modulus, per word}
    {{1.93, 0, 1.1, 7.4, 14}, {2.07, 0, 0.73, 3.2, 11}},        // tiles of a row
    {{1.49, 0.74, 1.2, 6.6, 14.5}, {1.56, 0.89, 0.92, 3.0, 11.5}},  // flattened, 16 positions
    {{2.93, 0.64, 2.6, 0, 20.5}, {2.49, 1.5, 1.95, 2.9, 13}},   // flattened, 32 positions
};
constexpr int kRowTiles = 0, kFlat16 = 1, kFlat32 = 2;

struct Form {
    int tiles;
    bool split;  // a workgroup per packed word
};

// With a workgroup per word on flattened tiles, every workgroup of one modulus
// and output channel group reads the same weights (37 KB a chunk) once per group
// of four residues.  Where the layer's weights (36 KB per modulus, chunk and
// group) exceed what an XCD's 4 MB L2 holds of them beside the planes, the groups
// are dealt to the XCDs so that one L2 serves a group.  32-position tiles wait for
// their weights and gain 4% on geometric mean from 7 MB on (49 of the 700 layers;
// 14x14 256 -> 256 189 -> 178 us, 512 -> 512 15%), and lose as much where the
// weights are few; 16-position tiles hold the next chunk's weights in registers
// and gain 2-3% on layers of few tiles with 8 groups (7x7 512 -> 512 208 -> 203
// us), else lose: a word's workgroups then no longer share plane lines in one L2
// (2 or 4 groups 2-3%, one group 17%).
bool deal_groups(int tiles, uint32_t k, uint32_t ncc, uint32_t ogroups) {
    const uint32_t weights = k * ncc * ogroups;  // in 36 KB
    if (tiles == kFlat16) return ogroups % kXcds == 0 && weights >= 384;
    return tiles == kFlat32 && (ogroups % kXcds == 0 || ogroups == 2 || ogroups == 4) && weights >= 192;
}

uint64_t form_tiles(const LinPlan &L, int tiles) {
    const uint64_t q = static_cast<uint64_t>(L.rows) * L.wp;
    return L.nimg * (tiles == kRowTiles ? static_cast<uint64_t>(L.rows) * ((L.cols + 15) / 16)
                     : tiles == kFlat16 ? (q + 15) / 16
                                        : (q + 31) / 32);
}

// L: rows, cols, wp, nimg, ncc and ogroups filled.
Form choose_form(const LinPlan &L, const redash_linear_params *p) {
    uint32_t pairs = 0, total = 0, most[2] = {0, 0};  // packed words, stages of a tile, of its longest workgroup
    for (uint32_t i = 0; i < p->k; ++i) {
        ModConst mc;
        fill_mod_const(p->moduli[i], &mc);
        const uint32_t full = (mc.g + 3) / 4, last = (mc.glast + 3) / 4, all = (mc.W - 1) * full + last;
        pairs += mc.W;
        total += all;
        if (all > most[0]) most[0] = all;
        if (full > most[1]) most[1] = full;
    }
    auto cost = [&](const Form &f) -> double {
        const FormCost &c = kFormCost[f.tiles][f.split];
        const double groups = static_cast<double>(form_tiles(L, f.tiles)) * L.ogroups;
        const double columns = f.tiles == kRowTiles ? 0 : (f.tiles == kFlat16 ? 16 : 32) + 2.0 * L.wp + 2;
        const double stages = groups * total * L.ncc, workgroups = groups * (f.split ? pairs : p->k);
        const double t = (stages * (c.stage + c.column * columns / 100) + workgroups * c.start) / 512 +
                         c.serial * most[f.split] * L.ncc + c.fixed;
        return f.split && deal_groups(f.tiles, p->k, L.ncc, L.ogroups) ? 0.95 * t : t;
    };
    // the simplest form unless another promises 2%: rows of at most 8 outputs
    // flattened, wider ones in row tiles
    Form best;
    best.tiles = L.cols <= 8 ? kFlat16 : kRowTiles;
    best.split = form_tiles(L, best.tiles) * p->k * L.ogroups < 2048;
    double least = cost(best) / 1.02;
    for (int tiles : {kRowTiles, kFlat16, kFlat32})
        for (bool split : {false, true}) {
            const double t = cost(Form{tiles, split});
            if (t < least) {
                least = t;
                best = Form{tiles, split};
            }
        }
    return best;
}

}  // namespace

int build_lin_plan(const redash_linear_params *p, LinPlan *L) {
    if (!p || !L) return REDASH_E_NULL;
    memset(L, 0, sizeof *L);
    if (p->k < 1 || p->k > static_cast<uint32_t>(kMaxK)) return REDASH_E_PARAM;
    unsigned __int128 P = 1;
    for (uint32_t i = 0; i < p->k; ++i) {
        const uint32_t m = p->moduli[i];
        if (!modulus_ok(m)) return REDASH_E_PARAM;
        if (i > 0 && m <= p->moduli[i - 1]) return REDASH_E_PARAM;
        for (uint32_t j = 0; j < i; ++j)
            if (gcd32(m, p->moduli[j]) != 1) return REDASH_E_PARAM;
        P *= m;
    }
    if (P >= (static_cast<unsigned __int128>(1) << 63)) return REDASH_E_PARAM;
    if (!p->batch || !p->c_in || !p->h_in || !p->w_in || !p->c_out || !p->kh || !p->kw || !p->stride)
        return REDASH_E_PARAM;
    if (p->pad >= p->kh || p->pad >= p->kw) return REDASH_E_PARAM;
    if (p->h_in + 2 * p->pad < p->kh || p->w_in + 2 * p->pad < p->kw) return REDASH_E_PARAM;
    const uint64_t taps = static_cast<uint64_t>(p->kh) * p->kw;
    if (taps > kLinMaxTaps || taps * p->c_in > kLinMaxK) return REDASH_E_PARAM;
    const uint32_t ho = (p->h_in + 2 * p->pad - p->kh) / p->stride + 1;
    const uint32_t wo = (p->w_in + 2 * p->pad - p->kw) / p->stride + 1;
    const uint64_t n_in = static_cast<uint64_t>(p->batch) * p->c_in * p->h_in * p->w_in;
    const uint64_t n_out = static_cast<uint64_t>(p->batch) * p->c_out * ho * wo;
    if (n_in >= (1ull << 30) || n_out >= (1ull << 30)) return REDASH_E_PARAM;

    L->k = p->k;
    L->c_in = p->c_in;
    L->c_out = p->c_out;
    L->kh = p->kh;
    L->kw = p->kw;
    L->stride = p->stride;
    L->pad = p->pad;
    L->n_in = n_in;
    L->n_out = n_out;
    const bool dense = p->h_in == 1 && p->w_in == 1 && p->kh == 1 && p->kw == 1;
    if (dense) {
        // (batch, c_in) row-major: the batch is the position axis of one image
        L->in_rows = 1;
        L->in_cols = p->batch;
        L->rows = 1;
        L->cols = p->batch;
        L->nimg = 1;
        L->sN = 0;
        L->sC = 1;
        L->sY = 0;
        L->sX = p->c_in;
        L->oN = 0;
        L->oO = 1;
        L->oY = 0;
        L->oX = p->c_out;
    } else {
        L->in_rows = p->h_in;
        L->in_cols = p->w_in;
        L->rows = ho;
        L->cols = wo;
        L->nimg = p->batch;
        L->sN = p->c_in * p->h_in * p->w_in;
        L->sC = p->h_in * p->w_in;
        L->sY = p->w_in;
        L->sX = 1;
        L->oN = p->c_out * ho * wo;
        L->oO = ho * wo;
        L->oY = wo;
        L->oX = 1;
    }
    L->taps = static_cast<uint32_t>(taps);
    // Column fold: with few input channels the kw columns of a kernel row
    // become kw c_in channels of a kh x 1 kernel, so that a K slice carries
    // kw c_in weights instead of c_in and up to 16 - c_in zeros (the 7x7
    // stride-2 stem over 3 channels: 4 K steps of 64 instead of 13).  The
    // planes stay unfolded, c_in bytes per position: the kw c_in bytes of a
    // window are consecutive there, and the staging loads them from the byte
    // where the window begins (the bytes after it meet zero weights), one
    // staged column per output column.  Where the staged halo of a 16-position
    // tile fits (16 kh 16-byte pieces per 16 of the chunk's 16, 32 or 64
    // channels).  From here on c_in, kw and taps are those of the folded layer.
    L->fold_c = 0;
    const uint32_t cf = p->kw * p->c_in, ckf = cf <= 16 ? 16u : cf <= 32 ? 32u : 64u;
    if (!dense && p->kw > 1 && p->c_in < 16 && cf <= 64 && p->kh * 16 * (ckf / 16) <= 2 * kLinBlock) {
        L->fold_c = p->c_in;
        L->c_in = p->kw * p->c_in;
        L->kw = 1;
        L->taps = p->kh;
    }
    // channel chunk: 64, or fewer when the channels are few or the taps many
    const uint32_t cin16 = round_up(L->c_in, 16);
    uint32_t ck = 64;
    while (ck > 16 && (ck / 2 >= cin16 || round_up(L->taps * ck, 64) > 1024)) ck /= 2;
    L->ck = ck;
    L->lg_ck = ck == 64 ? 6 : ck == 32 ? 5 : 4;
    L->kc = round_up(L->taps * ck, 64);
    L->ncc = (L->c_in + ck - 1) / ck;
    L->cp = L->fold_c ? L->fold_c : L->ncc * ck;
    L->hp = L->in_rows + 2 * p->pad;
    // (folded: up to the last window's end, so that a plane never takes more
    // than ck bytes for each column a window can begin at)
    L->wp = L->fold_c ? (L->cols - 1) * p->stride + p->kw : L->in_cols + 2 * p->pad;
    L->gstep = L->fold_c ? p->stride : 1;
    L->lstep = L->fold_c ? 1 : p->stride;
    L->xlast = L->fold_c ? (L->cols - 1) * p->stride : L->wp - 1;
    // M = ceil(2^16 / kw) <= 2^16: with e = M kw - 2^16 < kw, (t M) >> 16 =
    // floor(t/kw + t e / (kw 2^16)), and t e / 2^16 < 64 kw / 2^16 < 1 keeps
    // the error below 1/kw for every tap t < 64 and kw <= 64 (t M < 2^22: a
    // 24-bit multiply).  (2^32 / kw would not fit 32 bits for kw = 1.)
    L->kw_magic = ((1u << 16) + L->kw - 1) / L->kw;
    L->o_pad = round_up(p->c_out, kLinOTile);
    L->ogroups = L->o_pad / kLinOTile;
    // 16-byte LDS reads of 16 rows (or columns) at a stride of S bytes, four
    // 16-byte chunks each, run without bank conflicts on this LDS when
    // S / 16 = 2 mod 4 (measured: 96, 160, 224, 608 are conflict-free; 80,
    // 112, 128, 592 are not).  Weight rows: kc is a multiple of 64, so kc + 32.
    L->astride = L->kc + 32;
    L->lds_a = kLinOTile * L->astride;
    // Staged input: per residue kh rows of xw columns of ck channel bytes,
    // columns padded to xstride.  A fragment reads 16 columns conv-stride
    // apart: with 64-channel chunks the padding makes stride * xstride / 16
    // = 2 mod 4 where it can (odd strides: 96 bytes; strides 2 mod 4: 80).
    // 16-byte LDS writes go 8 lanes per cycle over 32 banks: the 8 lanes of
    // a write group take two columns wpair apart so that their 4 chunks each
    // fall in distinct bank groups (xstride / 16 = 6: 2 apart; 5: 4 apart).
    if (ck == 64) {
        L->xstride = (L->lstep % 2 == 1) ? 96 : 80;
        L->wpair = L->xstride == 96 ? 2 : 4;
    } else {
        // (folded, 32 channels: the two chunks of 16 columns fill 512 bytes)
        L->xstride = ck == 16 ? 16 : L->fold_c ? ck : ck + 16;
        L->wpair = 1;
    }
    // tile width: 32 or 16 positions, no wider than the row needs (64 would
    // not fit the registers of two waves per SIMD), and at most 512 staged
    // 16-byte pieces per residue (two per thread)
    L->xt = 32;
    while (L->xt > 16 && L->xt / 2 >= L->cols) L->xt /= 2;
    auto pieces = [&](uint32_t xt) { return L->kh * ((xt - 1) * L->lstep + L->kw) * (ck / 16); };
    if (L->xt == 32 && pieces(32) > 2 * kLinBlock) L->xt = 16;
    // a folded layer's few K steps leave a wave waiting for its staging and
    // epilogue: 16-position tiles (122 VGPRs, 33 KB of LDS) run four waves per
    // SIMD instead of two (7x7 stem 0.298 -> 0.224 ms)
    if (L->fold_c) L->xt = 16;
    // a 3x3 kernel over several 64-channel chunks keeps the next chunk's
    // weights in registers, which only the 16-position tile has room for
    if (L->ncc > 1 && ck == 64 && p->kh == 3 && p->kw == 3) L->xt = 16;
    if (pieces(L->xt) > 2 * kLinBlock) return REDASH_E_PARAM;
    L->xw = (L->xt - 1) * L->lstep + L->kw;
    L->halo = L->kh * L->xw * L->xstride;
    L->tile_rows = L->rows;
    // Flattened tiles (3x3, stride 1, several 64-channel chunks): output q =
    // y wp + x of the padded plane reads q + dy wp + dx, so a tile of XT
    // consecutive q stages one run of XT + 2 wp + 2 plane positions and reads
    // tap (dy, dx) at offset dy wp + dx; outputs with x >= cols are dropped at
    // the store.  Rows narrower than a tile leave no matrix columns idle that
    // way, and the staged run of a 32-position tile fits two workgroups per CU
    // up to 38 plane columns: a stage's weights (36 KB for four residues and a
    // chunk) then serve twice the positions.  (64 positions do not fit the
    // registers: 388 bytes of scratch.)  Which form: choose_form.
    L->flat = 0;
    const bool several33 = p->stride == 1 && L->kh == 3 && L->kw == 3 && ck == 64 && L->ncc > 1 && L->wp <= 38;
    Form form{kRowTiles, false};
    if (several33) form = choose_form(*L, p);
    if (form.tiles != kRowTiles) {
        L->flat = 1;
        L->xt = form.tiles == kFlat32 ? 32 : 16;
        L->xw = L->xt + 2 * L->wp + 2;
        L->halo = L->xw * L->xstride;
        L->tile_rows = 1;
        if (L->xw * (ck / 16) > 2 * kLinBlock) return REDASH_E_PARAM;  // not reached: at most 110 columns
    }
    L->ostride = L->xt + 4;  // the four lane groups of an atomic OR fall 16 banks apart
    L->lds_b = 4 * L->halo;
    // the merged output words overlay the staged inputs (used at the end of
    // a packed word, after every wave has read its fragments)
    L->lds_o = kLinOTile * L->ostride * 4;
    // then the accumulator seeds of the 64 output channels (base, -b mod m)
    L->lds_bytes = L->lds_a + (L->lds_b > L->lds_o ? L->lds_b : L->lds_o) + 2 * kLinOTile * 4;
    if (L->lds_bytes > kLinMaxLds) return REDASH_E_PARAM;
    L->xtiles = (L->flat ? L->rows * L->wp + L->xt - 1 : L->cols + L->xt - 1) / L->xt;
    L->plane_bytes = static_cast<uint64_t>(L->nimg) * L->hp * L->wp * L->cp;
    // folded: the last window's pieces are read past the last position (c_in
    // is kw times the layer's own), and whole words are written
    if (L->fold_c) L->plane_bytes = (L->plane_bytes + (ck - L->c_in) + 15) / 16 * 16;
    if (L->plane_bytes >= (1ull << 32)) return REDASH_E_PARAM;  // 32-bit offsets within a plane

    uint32_t woff = 0, pl_off = 0, np = 0;
    for (uint32_t i = 0; i < p->k; ++i) {
        ModConst mc;
        fill_mod_const(p->moduli[i], &mc);
        LinMod &lm = L->mod[i];
        lm.m = mc.m;
        lm.b = mc.b;
        lm.g = mc.g;
        lm.W = mc.W;
        lm.glast = mc.glast;
        lm.woff = woff;
        lm.pl_off = pl_off;
        lm.bp = mc.b == 1 ? 1u : mc.b == 2 ? 2u : mc.b <= 4 ? 4u : 8u;
        const uint32_t f = 8 / lm.bp;
        lm.lgf = f == 8 ? 3u : f == 4 ? 2u : f == 2 ? 1u : 0u;
        lm.ppw = (mc.g + f - 1) / f;
        lm.rep = f > 1 ? ((1u << lm.bp) - 1u) * 0x01010101u : 0xffffffffu;
        woff += mc.W;
        pl_off += (mc.W - 1) * lm.ppw + (mc.glast + f - 1) / f;
        // |sum w v| <= K floor(m/2) (m - 1) =: B (signed weights, residues v < m);
        // u = sum w v + off (+ (-b mod m) R_j, below m^2) lies in [0, 2B + m^2),
        // below 2^31 for K <= 16384, and u / m < 2^23 (a signed 24-bit product)
        const uint64_t K = static_cast<uint64_t>(L->taps) * L->c_in;
        const uint64_t B = K * (mc.m / 2) * (mc.m - 1);
        lm.off = static_cast<uint32_t>((B + mc.m - 1) / mc.m * mc.m);
        const uint64_t u_max = lm.off + B + static_cast<uint64_t>(mc.m) * mc.m;
        if (u_max >= (1ull << 31) || u_max / mc.m >= (1ull << 23)) return REDASH_E_PARAM;
        if (u_max * mc.m < (1ull << 32)) {
            lm.divM = static_cast<uint32_t>(((1ull << 32) + mc.m - 1) / mc.m);  // exact: u m < 2^32
            lm.divS = 0;
        } else {
            uint32_t fix = 0;
            division_constants(mc.m, 1ull << 31, &lm.divM, &lm.divS, &fix);
            if (fix) return REDASH_E_PARAM;  // not reached: below 2^31 the round-up method is exact
        }
        for (uint32_t w = 0; w < mc.W; ++w) {
            if (np >= kLinMaxPairs) return REDASH_E_PARAM;
            L->pair_mod[np] = static_cast<uint8_t>(i);
            L->pair_word[np] = static_cast<uint8_t>(w);
            ++np;
        }
    }
    L->npairs = np;
    // A workgroup per packed word rather than per modulus (both contraction
    // kernels) when the per-modulus grid is small: the small moduli, with the
    // most residues (128 for m = 2, 25 for 37 at 128-bit labels), would
    // otherwise set the launch's length; measured slower on large grids,
    // where the chip is full either way.
    const uint64_t tiles = static_cast<uint64_t>(L->nimg) * L->tile_rows * L->xtiles;
    const uint64_t grid_mod = (L->ncc > 1 ? tiles : (tiles + 3) / 4) * L->k * L->ogroups;  // 4 tiles per workgroup
    L->word_split = several33 ? form.split : grid_mod < 2048;
    L->og_xcd = L->word_split && L->flat && deal_groups(form.tiles, L->k, L->ncc, L->ogroups) &&
                tiles * L->npairs * L->ogroups < (1u << 28);  // (a one-dimensional grid, up to 7 words more)
    L->total_planes = pl_off;
    L->rowsum_off = static_cast<uint64_t>(L->k) * L->ncc * L->o_pad * L->kc;
    return REDASH_OK;
}

uint64_t prepared_bytes(const LinPlan &L) { return L.rowsum_off + 4ull * L.k * L.o_pad; }

uint64_t work_bytes(const LinPlan &L) { return static_cast<uint64_t>(L.total_planes) * L.plane_bytes; }

uint32_t total_words(const LinPlan &L) {
    uint32_t t = 0;
    for (uint32_t i = 0; i < L.k; ++i) t += L.mod[i].W;
    return t;
}

}  // namespace redash
