// Garbled linear layers (dense, 2-D convolution) on LabelTensors for gfx950.
//
// With public integer weights, a linear layer is free label arithmetic
// (Sec. 2.3): Y_o = sum_j w_oj X_j mod m, residue by residue, and the garbler
// sets Z_o = sum_j w_oj Z_j - b_o R.  Every residue of every label is an
// independent convolution with the same weights, so the layer is one dense
// integer contraction per (modulus, residue): int8 matrix cores do it.
//
//   * A weight acts through its residue mod m; reduced into the signed range
//     of Z_m it fits a signed byte for every m <= 255 (|w| <= 127).
//   * A residue v < m <= 128 is a valid signed byte as it is; for m > 128 it
//     enters as v - 128 (v XOR 0x80), and adding 128 * sum_k w (the row sums,
//     prepared with the weights) restores sum w v exactly.
//
// Two kernels per call, as the host plan (linear_plan.cpp) says:
//   k_linear_unpack  reads the packed input labels once and writes every
//                    residue as a byte (or a field of one, for the small
//                    moduli) into residue planes in the caller's working
//                    buffer, one plane per residue for every input position,
//                    channel-last with the zero padding already in place, so
//                    that a 16-byte load gives a matrix-core fragment of 16
//                    channels (HBM-bound); k_linear_unpack_rows does so for a
//                    layer of few channels, without gaps between positions;
//   k_linear_gemm_w  (one channel chunk) per workgroup: one modulus (or packed
//                    word) and 64 output channels, the weights staged in LDS
//                    once; each wave then takes its own row segment of XT (32
//                    or 16) output positions, 4 x (XT/16) MFMA 16x16x64 tiles,
//                    and runs through every residue with its own staged input
//                    halo, reducing the int32 sums mod m into PK32 fields and
//                    storing each packed word whole;
//   k_linear_gemm    (several channel chunks) per workgroup: one modulus (or
//                    packed word), 64 output channels and a tile of a row or of
//                    the flattened plane; wave q takes residue j0 + q of each
//                    packed word, the halos and the weights of each chunk staged
//                    by the workgroup, the residues of a word merged across the
//                    waves in LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/redash.h"
#include "linear_plan.hpp"

namespace redash {

// ---------------------------------------------------------------------------
// Weight preparation.
// Prepared layout: for modulus i, channel chunk cc, output channel o < o_pad:
// kc bytes, byte tap * ck + c_local = the weight w[o][cc ck + c_local][tap]
// reduced into the signed range of Z_m (0 beyond c_out, c_in or the taps).
// Then int32 row sums sum_{c, tap} of those values, [i][o].
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t signed_residue(int32_t w, uint32_t m) {
    int32_t r = w % static_cast<int32_t>(m);
    if (r < 0) r += static_cast<int32_t>(m);
    return r >= static_cast<int32_t>((m + 1) / 2) ? r - static_cast<int32_t>(m) : r;
}

__global__ void __launch_bounds__(256) k_linear_prepare(const LinPlan L, const int32_t *__restrict__ wts,
                                                        uint8_t *__restrict__ prep) {
    const uint64_t total = L.rowsum_off;
    for (uint64_t e = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; e < total;
         e += static_cast<uint64_t>(gridDim.x) * 256) {
        const uint32_t kb = static_cast<uint32_t>(e % L.kc);
        uint64_t r = e / L.kc;
        const uint32_t o = static_cast<uint32_t>(r % L.o_pad);
        r /= L.o_pad;
        const uint32_t cc = static_cast<uint32_t>(r % L.ncc);
        const uint32_t i = static_cast<uint32_t>(r / L.ncc);
        const uint32_t tap = kb / L.ck, c = cc * L.ck + kb % L.ck;
        int32_t v = 0;
        if (o < L.c_out && c < L.c_in && tap < L.taps) {
            // folded: channel c = dx c_in' + c' of kernel row tap is weight
            // (o, c', tap, dx) of the layer's kh x kw kernel (kw = c_in / c_in')
            const uint32_t kw0 = L.fold_c ? L.c_in / L.fold_c : 1u;
            const uint64_t at = L.fold_c ? (static_cast<uint64_t>(o) * L.fold_c + c % L.fold_c) * (L.taps * kw0) +
                                               static_cast<uint64_t>(tap) * kw0 + c / L.fold_c
                                         : (static_cast<uint64_t>(o) * L.c_in + c) * L.taps + tap;
            v = signed_residue(wts[at], L.mod[i].m);
        }
        prep[e] = static_cast<uint8_t>(static_cast<int8_t>(v));
    }
}

__global__ void __launch_bounds__(256) k_linear_rowsums(const LinPlan L, const int32_t *__restrict__ wts,
                                                        uint8_t *__restrict__ prep) {
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= L.k * L.o_pad) return;
    const uint32_t i = e / L.o_pad, o = e % L.o_pad;
    int32_t s = 0;
    if (o < L.c_out)
        for (uint32_t c = 0; c < L.c_in; ++c)
            for (uint32_t t = 0; t < L.taps; ++t)
                s += signed_residue(wts[(static_cast<uint64_t>(o) * L.c_in + c) * L.taps + t], L.mod[i].m);
    reinterpret_cast<int32_t *>(prep + L.rowsum_off)[e] = s;
}

// ---------------------------------------------------------------------------
// Residue planes.  Plane pl_off_i + pn(w, j) (see LinMod) holds plane_bytes
// bytes: position (img, yp, xp) of the zero-padded input at
// ((img hp + yp) wp + xp) cp, its cp channel bytes after it.  A byte holds f
// residues of a modulus m <= 16 in bp-bit fields, or one residue v (16 < m <=
// 128) or v XOR 0x80 (m > 128); padding holds the byte of v = 0, channels
// past c_in meet zero weights.
// ---------------------------------------------------------------------------

// A word at byte offset `off` (below 2^32) of a uniform base: the offset stays
// a 32-bit VGPR next to a scalar base address.
__device__ __forceinline__ uint32_t load_word(const uint32_t *base, uint32_t off) {
    asm("" : "+v"(off));
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(base) + off);
}

typedef int32_t v4i __attribute__((ext_vector_type(4)));

// (from any byte: the pieces of a folded layer begin where their window does)
__device__ __forceinline__ v4i load16(const uint8_t *base, uint32_t off) {
    typedef int32_t v4i_any __attribute__((ext_vector_type(4), aligned(1)));
    asm("" : "+v"(off));
    return *reinterpret_cast<const v4i_any *>(base + off);
}

// Byte of plane h (of those of its packed word) for the word wd.
__device__ __forceinline__ uint32_t plane_byte(uint32_t wd, const LinMod &M, uint32_t h) {
    if (M.lgf == 0) return __builtin_amdgcn_ubfe(wd, M.b * h, M.b);     // one residue
    if (M.bp == M.b) return __builtin_amdgcn_ubfe(wd, 8 * h, 8);        // f adjacent fields, as in the word
    // b = 3: residues 2h and 2h + 1 into 4-bit fields
    return __builtin_amdgcn_ubfe(wd, 6 * h, 3) | (__builtin_amdgcn_ubfe(wd, 6 * h + 3, 3) << 4);
}

// A workgroup takes 64 padded positions and one 64-channel chunk of a packed
// word.  Loads: thread (p, c16) = (tid % 64, tid / 64) reads 16 channel words
// of position p, so each load instruction reads 64 consecutive positions of
// one channel plane; the words go through LDS ([position][channel], rows
// padded to 68 words).  Stores: thread (p, c16) = (tid / 4, tid % 4) writes
// the 16-byte piece of position p, channels 16 c16.., of every residue of the
// word: consecutive threads write consecutive pieces.
__global__ void __launch_bounds__(256) k_linear_unpack(const LinPlan L, const uint32_t *__restrict__ in,
                                                       uint8_t *__restrict__ planes) {
    __shared__ __align__(16) uint32_t T[64 * 68];
    // workgroups go round-robin to the XCDs by linear index: remap so that
    // each XCD takes runs of RUN neighbouring position blocks, the 8 XCDs
    // working on 8 neighbouring runs, so that most lines that neighbouring
    // blocks share (input rows are not line-aligned) are fetched into one L2
    // (one contiguous range per XCD fetches the fewest lines but streams
    // from HBM more slowly: 0.73 ms against 0.51)
    const uint32_t nx = gridDim.x, ny = gridDim.y, nt = nx * ny * gridDim.z;
    const uint32_t lin = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    constexpr uint32_t RUN = 16;
    const uint32_t full = nt / (kXcds * RUN) * (kXcds * RUN);
    const uint32_t lg = lin < full ? lin / (kXcds * RUN) * (kXcds * RUN) + (lin % kXcds) * RUN + (lin / kXcds) % RUN : lin;
    const uint32_t bx = lg % nx, by = (lg / nx) % ny, bz = lg / (nx * ny);
    const uint32_t pair = by;
    const uint32_t i = L.pair_mod[pair], w = L.pair_word[pair];
    const LinMod M = L.mod[i];
    const uint32_t g = (w + 1 == M.W) ? M.glast : M.g;
    const uint32_t tid = threadIdx.x;
    const uint32_t npos = L.nimg * L.hp * L.wp;
    const uint32_t pp0 = bx * 64, cbase = 64 * bz;
    const uint32_t ngrp = (L.cp - cbase) / 16 < 4 ? (L.cp - cbase) / 16 : 4u;  // 16-channel groups of this chunk
    const uint32_t flip = M.m > 128 ? 0x80808080u : 0u;
    // position of (padded) index pp: inside the input, and the word offset there
    auto at = [&](uint32_t pp, bool &inside) -> uint32_t {
        const uint32_t xp = pp % L.wp, t = pp / L.wp;
        const uint32_t yp = t % L.hp, img = t / L.hp;
        const int32_t y = static_cast<int32_t>(yp) - static_cast<int32_t>(L.pad);
        const int32_t x = static_cast<int32_t>(xp) - static_cast<int32_t>(L.pad);
        inside = y >= 0 && y < static_cast<int32_t>(L.in_rows) && x >= 0 && x < static_cast<int32_t>(L.in_cols);
        return inside ? (img * L.sN + static_cast<uint32_t>(y) * L.sY + static_cast<uint32_t>(x) * L.sX) * 4u : 0u;
    };
    {
        const uint32_t p = tid % 64, c16 = tid / 64, pp = pp0 + p;
        if (pp < npos && c16 < ngrp) {
            bool inside = false;
            const uint32_t a0 = at(pp, inside);
            const uint32_t *src = in + (static_cast<uint64_t>(M.woff) + w) * L.n_in;
            const uint32_t step = L.sC * 4u;
            const uint32_t c0 = cbase + 16 * c16;
            // padding reads position (0, 0) channel 0, channels past c_in the
            // last channel: masked below
            const bool live = inside && c0 < L.c_in;
            const uint32_t cb = live ? c0 : 0u, last = live ? L.c_in - 1 - c0 : 0u;
            v4i q4[4];
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t q = static_cast<uint32_t>(4 * d + k);
                    q4[d][k] = static_cast<int32_t>(load_word(src, a0 + (cb + (q < last ? q : last)) * step));
                }
#pragma unroll
            for (int d = 0; d < 4; ++d) *reinterpret_cast<v4i *>(&T[p * 68 + 16 * c16 + 4 * d]) = q4[d];
        }
    }
    __syncthreads();
    const uint32_t p = tid / 4, c16 = tid % 4, pp = pp0 + p;
    if (pp >= npos || c16 >= ngrp) return;  // no barrier follows
    bool inside = false;
    (void)at(pp, inside);
    const uint32_t c0 = cbase + 16 * c16;
    uint32_t wd[16];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const v4i v = *reinterpret_cast<const v4i *>(&T[p * 68 + 16 * c16 + 4 * d]);
#pragma unroll
        for (int k = 0; k < 4; ++k) wd[4 * d + k] = static_cast<uint32_t>(v[k]);
    }
    const uint32_t nlive = !inside || c0 >= L.c_in ? 0u : (L.c_in - c0 < 16 ? L.c_in - c0 : 16u);  // live channels
    uint8_t *dst = planes + static_cast<uint64_t>(M.pl_off + w * M.ppw) * L.plane_bytes + static_cast<uint64_t>(pp) * L.cp + c0;
    const uint32_t nplanes = (g + (1u << M.lgf) - 1) >> M.lgf;
    for (uint32_t h = 0; h < nplanes; ++h) {
        v4i v;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t y = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t q = static_cast<uint32_t>(4 * d + k);
                const uint32_t x = plane_byte(wd[q], M, h);
                y |= (q < nlive ? x : 0u) << (8 * k);
            }
            v[d] = static_cast<int32_t>(y ^ flip);
        }
        *reinterpret_cast<v4i *>(dst + static_cast<uint64_t>(h) * L.plane_bytes) = v;
    }
}

// The planes of a folded layer (few channels): c_in bytes per padded position,
// without gaps.  A thread writes four consecutive bytes of every residue of a
// packed word.  (The folded planes that this replaces held every window on its
// own, 7.7 times the bytes for the 7x7 stem: 0.222 ms of unpacking.)
__global__ void __launch_bounds__(256) k_linear_unpack_rows(const LinPlan L, const uint32_t *__restrict__ in,
                                                            uint8_t *__restrict__ planes) {
    const uint32_t pair = blockIdx.y;
    const uint32_t i = L.pair_mod[pair], w = L.pair_word[pair];
    const LinMod M = L.mod[i];
    const uint32_t g = (w + 1 == M.W) ? M.glast : M.g;
    const uint32_t flip = M.m > 128 ? 0x80808080u : 0u;
    const uint32_t total = L.nimg * L.hp * L.wp * L.cp;  // below 2^32 (plane_bytes is)
    const uint32_t b0 = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (b0 >= total) return;
    const uint32_t *src = in + (static_cast<uint64_t>(M.woff) + w) * L.n_in;
    uint32_t wd[4];
    uint32_t pos = b0 / L.cp, c = b0 - pos * L.cp;
    uint32_t xp = pos % L.wp, t = pos / L.wp;
    uint32_t yp = t % L.hp, img = t / L.hp;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int32_t y = static_cast<int32_t>(yp) - static_cast<int32_t>(L.pad);
        const int32_t x = static_cast<int32_t>(xp) - static_cast<int32_t>(L.pad);
        const bool inside = img < L.nimg && y >= 0 && y < static_cast<int32_t>(L.in_rows) && x >= 0 &&
                            x < static_cast<int32_t>(L.in_cols);
        const uint32_t at =
            img * L.sN + c * L.sC + static_cast<uint32_t>(y) * L.sY + static_cast<uint32_t>(x) * L.sX;
        wd[k] = inside ? src[at] : 0u;
        // the next byte: channel, column, row, image
        if (++c == L.cp) {
            c = 0;
            if (++xp == L.wp) {
                xp = 0;
                if (++yp == L.hp) yp = 0, ++img;
            }
        }
    }
    uint8_t *dst = planes + static_cast<uint64_t>(M.pl_off + w * M.ppw) * L.plane_bytes + b0;
    const uint32_t nplanes = (g + (1u << M.lgf) - 1) >> M.lgf;
    for (uint32_t h = 0; h < nplanes; ++h) {
        uint32_t y = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) y |= plane_byte(wd[k], M, h) << (8 * k);
        *reinterpret_cast<uint32_t *>(dst + static_cast<uint64_t>(h) * L.plane_bytes) = y ^ flip;
    }
}

// Residue j's values from a 16-byte piece of its plane: field j mod f of
// every byte (f > 1), or the bytes themselves.
__device__ __forceinline__ v4i plane_field(const v4i &v, const LinMod &M, uint32_t j) {
    if (M.lgf == 0) return v;
    const uint32_t sh = M.bp * (j & ((1u << M.lgf) - 1u));
    v4i r;
#pragma unroll
    for (int d = 0; d < 4; ++d) r[d] = static_cast<int32_t>((static_cast<uint32_t>(v[d]) >> sh) & M.rep);
    return r;
}

// ---------------------------------------------------------------------------
// The contraction.
// ---------------------------------------------------------------------------
// At least two waves per SIMD; without K33, on 16-position tiles, the registers
// and the LDS allow three (1x1 256 -> 512 stride 2 at 14x14 0.121 -> 0.094 ms).
// With K33 only two fit, and the upper bound lets the compiler schedule for two
// (3x3 stride 2 256 -> 512 at 14x14 202 -> 198.5 us, on a short base batch 8
// 197.5 -> 194.0).
// K33 (> 0): a 3x3 kernel with 64-channel chunks (taps = K steps, kc = 576)
// and K33 bytes per staged column, the K loop unrolled with every fragment
// offset known but the row stride; 0: any kernel.  DEALT: the grid of og_xcd, a
// form of its own: the mapping's divisions at every workgroup's start cost the
// other layers up to 2% (1x1 256 -> 512 at 28x28, batch 8, on a short base 494 ->
// 485 us without them).
template <int NCB, bool GARBLE, int K33, bool DEALT>
__global__ void __launch_bounds__(kLinBlock) __attribute__((amdgpu_waves_per_eu(2, K33 > 0 ? 2 : 8)))
k_linear_gemm(const LinPlan L, const uint8_t *__restrict__ planes, const uint8_t *__restrict__ prep,
              const int64_t *__restrict__ bias, const uint32_t *__restrict__ offsets, uint32_t *__restrict__ out) {
    extern __shared__ __align__(16) uint8_t lds[];
    uint8_t *Al = lds;
    uint8_t *Bl = lds + L.lds_a;
    uint32_t *Ol = reinterpret_cast<uint32_t *>(lds + L.lds_a);  // overlays Bl

    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // consecutive tiles (neighbouring output rows, which share input rows) on
    // one XCD, whose L2 then serves the shared plane rows
    const uint32_t nb = gridDim.x, full = nb / kXcds * kXcds;
    uint32_t tile = blockIdx.x < full ? (blockIdx.x % kXcds) * (nb / kXcds) + blockIdx.x / kXcds : blockIdx.x;
    // one packed word (pair table entry blockIdx.z, the output channel group
    // blockIdx.y: the words of the small moduli, with the most residues, are
    // dispatched first for every group) or every word of modulus blockIdx.y
    uint32_t pair = blockIdx.z, og = L.word_split ? blockIdx.y : blockIdx.z;
    if constexpr (DEALT) {
        // workgroup 8 s + x runs on XCD x: its s-th (word, tile)
        const uint32_t x = blockIdx.x % kXcds, sl = blockIdx.x / kXcds;
        const uint32_t tiles = L.nimg * L.tile_rows * L.xtiles, t = sl / tiles;
        tile = sl - t * tiles;
        if (L.ogroups >= kXcds) {
            const uint32_t per = L.ogroups / kXcds;
            pair = t / per;
            og = x + kXcds * (t - pair * per);
        } else {
            const uint32_t share = kXcds / L.ogroups;
            og = x / share;
            pair = x % share + share * t;
        }
        if (pair >= L.npairs) return;  // (the whole workgroup, before any barrier)
    }
    const uint32_t i = L.word_split ? L.pair_mod[pair] : blockIdx.y;
    const uint32_t xtile = tile % L.xtiles;
    const uint32_t row = (tile / L.xtiles) % L.tile_rows;
    const uint32_t img = tile / (L.xtiles * L.tile_rows);
    const LinMod M = L.mod[i];
    const uint32_t w_lo = L.word_split ? L.pair_word[pair] : 0u;
    const uint32_t w_hi = L.word_split ? w_lo + 1 : M.W;
    constexpr uint32_t XT = 16 * NCB;
    const uint32_t x0 = xtile * XT;
    const int32_t *rowsum = reinterpret_cast<const int32_t *>(prep + L.rowsum_off) + i * L.o_pad + og * kLinOTile;
    const uint32_t ksteps = L.kc / 64;
    const uint32_t kg = 16 * (lane / 16);
    // staged bytes between kernel rows: a row of the halo, or wp positions of the flattened run
    const uint32_t rowb = (L.flat ? L.wp : L.xw) * L.xstride;

    // output channel of element r of row block ob for this lane
    auto o_local = [&](int ob, int r) -> uint32_t { return ob * 16 + 4 * (lane / 16) + r; };

    // The accumulators start at base = 128 rowsum (m > 128) + off (+ (-b mod
    // m) R_j for the garbler) and end at u = sum w v + off (+ ...) in
    // [0, 2^31) with u / m < 2^23.  The 64 output channels' base and -b mod m
    // sit in LDS after the staging area (read at each residue's first chunk).
    uint32_t *sbase = reinterpret_cast<uint32_t *>(lds + L.lds_bytes - 2 * kLinOTile * 4);
    uint32_t *snegb = sbase + kLinOTile;
    if (tid < kLinOTile) {
        const bool shifted = M.m > 128;
        sbase[tid] = (shifted ? static_cast<uint32_t>(128 * rowsum[tid]) : 0u) + M.off;
        uint32_t nb = 0;
        if constexpr (GARBLE) {
            const uint32_t o = og * kLinOTile + tid;
            if (bias && o < L.c_out) {
                int64_t bm = bias[o] % static_cast<int64_t>(M.m);
                if (bm < 0) bm += M.m;
                nb = (M.m - static_cast<uint32_t>(bm)) % M.m;
            }
        }
        snegb[tid] = nb;
    }
    __syncthreads();

    // This thread's (at most two) staged pieces: piece e = tid + 256 t of a
    // residue's halo is (row dy, column xin, 16 channels c16); its plane
    // offset (the column clamped into the padded row: the columns past the
    // row feed outputs that are dropped) and its LDS offset.
    const uint32_t c16n = L.ck / 16;
    const uint32_t pieces = (L.flat ? 1u : L.kh) * L.xw * c16n;
    uint32_t poff[2], loff[2];
    bool pval[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint32_t e = tid + t * kLinBlock;
        pval[t] = e < pieces;
        const uint32_t ee = pval[t] ? e : 0u;
        const uint32_t c16 = ee % c16n, dy = ee / (c16n * L.xw);
        // column of this piece: within each full group of 2 wpair columns,
        // write slot j takes column j / 2 + (j % 2) wpair (a bijection)
        uint32_t xin = (ee / c16n) % L.xw;
        const uint32_t grp = 2 * L.wpair, gb = xin - xin % grp;
        if (gb + grp <= L.xw) xin = gb + (xin - gb) / 2 + ((xin - gb) % 2) * L.wpair;
        uint32_t xp = x0 * L.stride + xin;
        const uint32_t xlim = L.flat ? L.hp * L.wp : L.wp;  // flattened: the image's last position
        xp = xp < xlim ? xp : xlim - 1;
        poff[t] = ((img * L.hp + row * L.stride + dy) * L.wp + xp) * L.cp + 16 * c16;
        loff[t] = dy * rowb + xin * L.xstride + 16 * c16;
    }
    // fragment columns of this lane in the staged rows (tile column cb)
    uint32_t colb[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) colb[cb] = (cb * 16 + lane % 16) * L.stride * L.xstride;

    // Stages (w, j0, cc) in order: packed word, group of four residues,
    // channel chunk.  The pieces of the next stage are loaded into registers
    // while the current stage computes.
    struct Stage {
        uint32_t w, j0, cc;
    };
    auto g_of = [&](uint32_t w) { return (w + 1 == M.W) ? M.glast : M.g; };
    auto advance = [&](Stage &st) {
        if (++st.cc == L.ncc) {
            st.cc = 0;
            st.j0 += 4;
            if (st.j0 >= g_of(st.w)) {
                st.j0 = 0;
                ++st.w;
            }
        }
    };
    auto load_stage = [&](v4i (&pf)[2][4], const Stage &st) {
        const uint32_t g = g_of(st.w);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t j = st.j0 + q < g ? st.j0 + q : 0u;
            const uint8_t *plane =
                planes + static_cast<uint64_t>(M.pl_off + st.w * M.ppw + (j >> M.lgf)) * L.plane_bytes;
#pragma unroll
            for (int t = 0; t < 2; ++t) pf[t][q] = load16(plane, pval[t] ? poff[t] + st.cc * L.ck : 0u);
        }
    };

    uint32_t part[4][NCB][4];
    v4i acc[4][NCB];
    bool a_staged = false;
    Stage cur{w_lo, 0, 0}, ahead{w_lo, 0, 0};
    v4i pfA[2][4];
    load_stage(pfA, ahead);
    advance(ahead);
    // 3x3 kernels on 64-channel chunks (kc = 576: 64 rows of 36 16-byte
    // pieces, 9 per thread): the next chunk's weights are loaded into
    // registers while the current stage computes, as the input pieces are
    constexpr bool kWpf = K33 > 0 && NCB == 1;  // with 32-position tiles the registers do not suffice
    constexpr int kWq = kWpf ? 9 : 1;
    v4i wf[kWq];
    auto load_weights = [&](uint32_t cc) {
        const uint8_t *ap = prep + ((static_cast<uint64_t>(i) * L.ncc + cc) * L.o_pad + og * kLinOTile) * L.kc;
#pragma unroll
        for (int q = 0; q < kWq; ++q) {
            const uint32_t e = tid + kLinBlock * q, rr = e / 36, p = e % 36;
            wf[q] = *reinterpret_cast<const v4i *>(ap + static_cast<uint64_t>(rr) * L.kc + 16 * p);
        }
    };
    if constexpr (kWpf) load_weights(0);

    // One stage with the pieces in pf; returns false after the last stage.
    auto stage = [&](v4i (&pf)[2][4]) -> bool {
        const uint32_t w = cur.w, j0 = cur.j0, cc = cur.cc;
        const uint32_t g = g_of(w);
        const uint32_t j = j0 + wave;  // this wave's residue
        if (j0 == 0 && cc == 0) {
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) part[ob][cb][r] = 0;
        }
        if (cc == 0) {
            uint32_t Rj = 0;
            if constexpr (GARBLE) Rj = (offsets[M.woff + w] >> (M.b * j)) & ((1u << M.b) - 1u);
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t b0 = static_cast<int32_t>(sbase[o_local(ob, r)] + snegb[o_local(ob, r)] * Rj);
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) acc[ob][cb][r] = b0;
                }
        }
        __syncthreads();  // the previous stage's fragments have been read
        if (L.ncc > 1 || !a_staged) {
            if constexpr (kWpf) {
                // weights of chunk cc from the registers, then the next chunk's
#pragma unroll
                for (int q = 0; q < kWq; ++q) {
                    const uint32_t e = tid + kLinBlock * q, rr = e / 36, p = e % 36;
                    *reinterpret_cast<v4i *>(Al + rr * L.astride + 16 * p) = wf[q];
                }
                if (L.ncc > 1) load_weights(cc + 1 < L.ncc ? cc + 1 : 0u);
            } else {
                // weights of chunk cc: 64 rows of kc bytes, 16 bytes per load
                const uint8_t *ap =
                    prep + ((static_cast<uint64_t>(i) * L.ncc + cc) * L.o_pad + og * kLinOTile) * L.kc;
                const uint32_t per_row = L.kc / 16;
                for (uint32_t e = tid; e < kLinOTile * per_row; e += kLinBlock) {
                    const uint32_t rr = e / per_row, q = e % per_row;
                    *reinterpret_cast<uint4 *>(Al + rr * L.astride + 16 * q) =
                        *reinterpret_cast<const uint4 *>(ap + static_cast<uint64_t>(rr) * L.kc + 16 * q);
                }
            }
            a_staged = true;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (j0 + q < g) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    if (pval[t]) *reinterpret_cast<v4i *>(Bl + q * L.halo + loff[t]) = plane_field(pf[t][q], M, j0 + q);
            }
        // pf is free: the next stage
        if (ahead.w < w_hi) load_stage(pf, ahead);
        advance(ahead);
        __syncthreads();
        if (j < g) {
            const uint8_t *Bw = Bl + wave * L.halo;
            if constexpr (K33 > 0) {
                // K step t is tap t = 3 dy + dx, the lane's 16 channels at kg
                const uint8_t *Ar = Al + (lane % 16) * (576 + 32) + kg;
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const uint8_t *Br = Bw + dy * rowb + kg;
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
                        const int kk = 3 * dy + dx;
                        v4i a[4];
#pragma unroll
                        for (int ob = 0; ob < 4; ++ob)
                            a[ob] = *reinterpret_cast<const v4i *>(Ar + ob * 16 * (576 + 32) + kk * 64);
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb) {
                            const v4i bf = *reinterpret_cast<const v4i *>(Br + colb[cb] + dx * K33);
#pragma unroll
                            for (int ob = 0; ob < 4; ++ob)
                                acc[ob][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[ob], bf, acc[ob][cb], 0, 0, 0);
                        }
                    }
                }
            } else {
                for (uint32_t kk = 0; kk < ksteps; ++kk) {
                    v4i a[4];
#pragma unroll
                    for (int ob = 0; ob < 4; ++ob)
                        a[ob] = *reinterpret_cast<const v4i *>(Al + (ob * 16 + lane % 16) * L.astride + kk * 64 + kg);
                    const uint32_t kidx = kk * 64 + kg;
                    uint32_t tap = kidx >> L.lg_ck;
                    if (tap >= L.taps) tap = 0;  // K padding: the weights there are 0
                    const uint32_t dy = __umul24(tap, L.kw_magic) >> 16, dx = tap - dy * L.kw;
                    const uint32_t boff = dy * rowb + dx * L.xstride + (kidx & (L.ck - 1u));
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const v4i bf = *reinterpret_cast<const v4i *>(Bw + boff + colb[cb]);
#pragma unroll
                        for (int ob = 0; ob < 4; ++ob)
                            acc[ob][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[ob], bf, acc[ob][cb], 0, 0, 0);
                    }
                }
            }
        }
        if (cc + 1 == L.ncc && j < g) {
            // epilogue of residue j: the residue of u mod m goes into the field
            const uint32_t sh = M.b * j;
            auto epilogue = [&](auto shifts) {
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const uint32_t u = static_cast<uint32_t>(acc[ob][cb][r]);
                            uint32_t q = __umulhi(u, M.divM);  // < 2^23
                            if constexpr (decltype(shifts)::value) q >>= M.divS;
                            const uint32_t res =
                                static_cast<uint32_t>(__mul24(static_cast<int32_t>(q), -static_cast<int32_t>(M.m))) + u;
                            part[ob][cb][r] |= res << sh;
                        }
            };
            if (M.divS == 0)
                epilogue(std::integral_constant<bool, false>{});
            else
                epilogue(std::integral_constant<bool, true>{});
        }
        advance(cur);
        if (cur.w != w) {
            // word w complete: merge the waves' fields (disjoint bits), store
            // whole words.  Ol overlays the staged inputs: every wave must be
            // done with its fragments first.
            __syncthreads();
            for (uint32_t e = tid; e < kLinOTile * L.ostride; e += kLinBlock) Ol[e] = 0;
            __syncthreads();
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (part[ob][cb][r])
                            atomicOr(&Ol[o_local(ob, r) * L.ostride + cb * 16 + lane % 16], part[ob][cb][r]);
            __syncthreads();
            uint32_t *dstp = out + (static_cast<uint64_t>(M.woff) + w) * L.n_out;
            for (uint32_t e = tid; e < kLinOTile * XT; e += kLinBlock) {
                const uint32_t ol = e / XT, xl = e % XT;
                const uint32_t o = og * kLinOTile + ol;
                uint32_t y = row, x = x0 + xl;
                if (L.flat) {
                    y = x / L.wp;
                    x -= y * L.wp;
                }
                if (o < L.c_out && x < L.cols && y < L.rows)
                    dstp[img * L.oN + o * L.oO + y * L.oY + x * L.oX] = Ol[ol * L.ostride + xl];
            }
        }
        return cur.w < w_hi;
    };
    while (stage(pfA)) {
    }
}

// ---------------------------------------------------------------------------
// The contraction for one channel chunk (ncc = 1), with independent waves.
// A workgroup stages the weights of its modulus and 64 output channels once;
// then each wave takes its own tile (one output row segment of XT positions,
// the 64 channels), stages its own input halo and runs through every residue
// of every packed word of the modulus in turn: MFMA over the halo, the next
// residue's halo written over it (LDS operations of a wave complete in
// order), the one after loaded into registers, the epilogue, and each packed
// word stored whole when its last residue is done.  No barrier after the
// weights are staged.
// ---------------------------------------------------------------------------
constexpr int kWavePieces = 8;  // staged 16-byte pieces per lane (a halo has at most 512)

// PL: staged pieces per lane (a 3x3 halo of 64-channel columns has at most 7 x 64)
template <int NCB, bool GARBLE, int K33, int PL>
__global__ void __launch_bounds__(kLinBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_linear_gemm_w(const LinPlan L, const uint8_t *__restrict__ planes, const uint8_t *__restrict__ prep,
                const int64_t *__restrict__ bias, const uint32_t *__restrict__ offsets, uint32_t *__restrict__ out) {
    extern __shared__ __align__(16) uint8_t lds[];
    uint8_t *Al = lds;
    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / 64);
    uint8_t *Bw = lds + L.lds_a + wave * L.halo;
    // accumulator seeds per output channel: 128 rowsum (m > 128) + off, and
    // for the garbler (-b mod m), to be multiplied by R_j
    int32_t *seed = reinterpret_cast<int32_t *>(lds + L.lds_a + 4 * L.halo);
    int32_t *negb = seed + kLinOTile;
    // one packed word (pair table entry blockIdx.z, output channel group
    // blockIdx.y) or every word of modulus blockIdx.y, as in k_linear_gemm
    const uint32_t i = L.word_split ? L.pair_mod[blockIdx.z] : blockIdx.y;
    const uint32_t og = L.word_split ? blockIdx.y : blockIdx.z;
    const LinMod M = L.mod[i];
    const uint32_t w_lo = L.word_split ? L.pair_word[blockIdx.z] : 0u;
    const uint32_t w_hi = L.word_split ? w_lo + 1 : M.W;
    if (tid < kLinOTile) {
        const int32_t *rs = reinterpret_cast<const int32_t *>(prep + L.rowsum_off) + i * L.o_pad + og * kLinOTile;
        seed[tid] = static_cast<int32_t>((M.m > 128 ? static_cast<uint32_t>(128 * rs[tid]) : 0u) + M.off);
        uint32_t nb = 0;
        if constexpr (GARBLE) {
            const uint32_t o = og * kLinOTile + tid;
            if (bias && o < L.c_out) {
                int64_t bm = bias[o] % static_cast<int64_t>(M.m);
                if (bm < 0) bm += M.m;
                nb = (M.m - static_cast<uint32_t>(bm)) % M.m;
            }
        }
        negb[tid] = static_cast<int32_t>(nb);
    }

    // weights of the one chunk: 64 rows of kc bytes
    {
        const uint8_t *ap = prep + (static_cast<uint64_t>(i) * L.o_pad + og * kLinOTile) * L.kc;
        const uint32_t per_row = L.kc / 16;
        for (uint32_t e = tid; e < kLinOTile * per_row; e += kLinBlock) {
            const uint32_t rr = e / per_row, q = e % per_row;
            *reinterpret_cast<uint4 *>(Al + rr * L.astride + 16 * q) =
                *reinterpret_cast<const uint4 *>(ap + static_cast<uint64_t>(rr) * L.kc + 16 * q);
        }
    }
    __syncthreads();  // the only barrier

    // this wave's tile; consecutive workgroups (neighbouring rows) on one XCD
    const uint32_t nb = gridDim.x, full = nb / kXcds * kXcds;
    const uint32_t blk = blockIdx.x < full ? (blockIdx.x % kXcds) * (nb / kXcds) + blockIdx.x / kXcds : blockIdx.x;
    const uint32_t tile = blk * 4 + wave;
    if (tile >= L.nimg * L.rows * L.xtiles) return;  // no barrier follows
    const uint32_t xtile = tile % L.xtiles;
    const uint32_t row = (tile / L.xtiles) % L.rows;
    const uint32_t img = tile / (L.xtiles * L.rows);
    constexpr uint32_t XT = 16 * NCB;
    const uint32_t x0 = xtile * XT;
    const uint32_t kg = 16 * (lane / 16);
    const uint32_t rowb = L.xw * L.xstride;
    auto o_local = [&](int ob, int r) -> uint32_t { return ob * 16 + 4 * (lane / 16) + r; };
    const bool full_tile = x0 + XT <= L.cols && (og + 1) * kLinOTile <= L.c_out;

    // staged pieces of this lane: piece e = lane + 64 s is (row dy, column,
    // 16 channels); plane offset (column clamped into the padded row) and LDS
    // offset (16 bits, 0xffff: not staged; two per register); the 8 lanes of
    // a write group take columns wpair apart
    const uint32_t c16n = L.ck / 16;
    const uint32_t pieces = L.kh * L.xw * c16n;
    uint32_t poff[PL], loff2[(PL + 1) / 2];
#pragma unroll
    for (int s = 0; s < (PL + 1) / 2; ++s) loff2[s] = 0;
#pragma unroll
    for (int s = 0; s < PL; ++s) {
        const uint32_t e = lane + 64 * s;
        const uint32_t ee = e < pieces ? e : 0u;
        const uint32_t c16 = ee % c16n, dy = ee / (c16n * L.xw);
        uint32_t xin = (ee / c16n) % L.xw;
        const uint32_t grp = 2 * L.wpair, gb = xin - xin % grp;
        if (gb + grp <= L.xw) xin = gb + (xin - gb) / 2 + ((xin - gb) % 2) * L.wpair;
        uint32_t xp = x0 * L.stride + xin * L.gstep;
        xp = xp < L.xlast ? xp : L.xlast;
        poff[s] = ((img * L.hp + row * L.stride + dy) * L.wp + xp) * L.cp + 16 * c16;
        const uint32_t lo = e < pieces ? dy * rowb + xin * L.xstride + 16 * c16 : 0xffffu;
        loff2[s / 2] |= lo << (16 * (s % 2));
    }
    auto loff = [&](int s) -> uint32_t { return (loff2[s / 2] >> (16 * (s % 2))) & 0xffffu; };
    uint32_t colb[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) colb[cb] = (cb * 16 + lane % 16) * L.lstep * L.xstride;

    // residue (w, j) (field j of packed word w) is in plane pn(w, j) of the
    // modulus; the halo of the next residue is staged after the operations
    // of this one from registers that hold its plane's pieces, and a plane
    // is loaded into them one residue before its first residue is staged
    auto g_of = [&](uint32_t w) { return (w + 1 == M.W) ? M.glast : M.g; };
    auto pn = [&](uint32_t w, uint32_t j) { return w * M.ppw + (j >> M.lgf); };
    v4i pf[PL];
    auto load = [&](uint32_t pl) {
        const uint8_t *plane = planes + static_cast<uint64_t>(M.pl_off + pl) * L.plane_bytes;
#pragma unroll
        for (int s = 0; s < PL; ++s) pf[s] = load16(plane, lane + 64 * s < pieces ? poff[s] : 0u);
    };
    auto stage = [&](uint32_t j) {
#pragma unroll
        for (int s = 0; s < PL; ++s)
            if (lane + 64 * s < pieces) *reinterpret_cast<v4i *>(Bw + loff(s)) = plane_field(pf[s], M, j);
    };
    load(pn(w_lo, 0));
    stage(0);
    // (nw, nj): the next residue to stage; its plane is in pf once staged
    uint32_t nw = w_lo, nj = 1;
    if (nj == g_of(w_lo)) nw = w_lo + 1, nj = 0;
    if (nw < w_hi && pn(nw, nj) != pn(w_lo, 0)) load(pn(nw, nj));

    uint32_t part[4][NCB][4];
    v4i acc[4][NCB];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[ob][cb][r] = 0;

    for (uint32_t w = w_lo; w < w_hi; ++w) {
        const uint32_t g = g_of(w);
        uint32_t Rw = 0;
        if constexpr (GARBLE) Rw = offsets[M.woff + w];
        for (uint32_t j = 0; j < g; ++j) {
            const int32_t Rj = GARBLE ? static_cast<int32_t>((Rw >> (M.b * j)) & ((1u << M.b) - 1u)) : 0;
            // the seeds of this lane's 4 output channels of each row block
            // (the C operand of the first K step)
            v4i b0[4];
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) {
                b0[ob] = *reinterpret_cast<const v4i *>(seed + ob * 16 + 4 * (lane / 16));
                if constexpr (GARBLE) b0[ob] += *reinterpret_cast<const v4i *>(negb + ob * 16 + 4 * (lane / 16)) * Rj;
            }
            if constexpr (K33 > 0) {
                // K step kk = 3 dy + dx; the fragments of step kk + 1 are
                // loaded before the matrix-core operations of step kk
                const uint8_t *Ar = Al + (lane % 16) * (576 + 32) + kg;
                auto frag = [&](int kk, v4i(&a)[4], v4i(&bq)[NCB]) {
#pragma unroll
                    for (int ob = 0; ob < 4; ++ob)
                        a[ob] = *reinterpret_cast<const v4i *>(Ar + ob * 16 * (576 + 32) + kk * 64);
                    const uint8_t *Br = Bw + (kk / 3) * rowb + kg + (kk % 3) * K33;
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) bq[cb] = *reinterpret_cast<const v4i *>(Br + colb[cb]);
                };
                auto mma = [&](int kk, const v4i(&a)[4], const v4i(&bq)[NCB]) {
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int ob = 0; ob < 4; ++ob)
                            acc[ob][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[ob], bq[cb], kk == 0 ? b0[ob] : acc[ob][cb],
                                                                                0, 0, 0);
                };
                v4i fa0[4], fb0[NCB], fa1[4], fb1[NCB];
                frag(0, fa0, fb0);
                // the wave's priority is raised while it issues its
                // matrix-core steps and lowered for the staging and epilogue
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int kk = 0; kk < 9; ++kk) {
                    // (scheduling barriers keep the loads of step kk + 1
                    // ahead of the operations of step kk)
                    if (kk % 2 == 0) {
                        if (kk + 1 < 9) frag(kk + 1, fa1, fb1);
                        __builtin_amdgcn_sched_barrier(0);
                        mma(kk, fa0, fb0);
                    } else {
                        if (kk + 1 < 9) frag(kk + 1, fa0, fb0);
                        __builtin_amdgcn_sched_barrier(0);
                        mma(kk, fa1, fb1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_s_setprio(0);
            } else {
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) acc[ob][cb] = b0[ob];
                const uint32_t ksteps = L.kc / 64;
                for (uint32_t kk = 0; kk < ksteps; ++kk) {
                    v4i a[4];
#pragma unroll
                    for (int ob = 0; ob < 4; ++ob)
                        a[ob] = *reinterpret_cast<const v4i *>(Al + (ob * 16 + lane % 16) * L.astride + kk * 64 + kg);
                    const uint32_t kidx = kk * 64 + kg;
                    uint32_t tap = kidx >> L.lg_ck;
                    if (tap >= L.taps) tap = 0;  // K padding: the weights there are 0
                    const uint32_t dy = __umul24(tap, L.kw_magic) >> 16, dx = tap - dy * L.kw;
                    const uint32_t boff = dy * rowb + dx * L.xstride + (kidx & (L.ck - 1u));
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const v4i bf = *reinterpret_cast<const v4i *>(Bw + boff + colb[cb]);
#pragma unroll
                        for (int ob = 0; ob < 4; ++ob)
                            acc[ob][cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[ob], bf, acc[ob][cb], 0, 0, 0);
                    }
                }
            }
            // the next residue's halo over this one (after this wave's reads,
            // in LDS order), then the plane of the one after into the
            // registers if it is a new plane
            if (nw < w_hi) {
                stage(nj);
                uint32_t mw = nw, mj = nj + 1;
                if (mj == g_of(mw)) mw += 1, mj = 0;
                if (mw < w_hi && pn(mw, mj) != pn(nw, nj)) load(pn(mw, mj));
                nw = mw;
                nj = mj;
            }
            // epilogue: residue of u mod m into field j
            const uint32_t sh = M.b * j;
            auto epilogue = [&](auto shifts) {
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const uint32_t u = static_cast<uint32_t>(acc[ob][cb][r]);
                            uint32_t q = __umulhi(u, M.divM);  // < 2^23
                            if constexpr (decltype(shifts)::value) q >>= M.divS;
                            const uint32_t res =
                                static_cast<uint32_t>(__mul24(static_cast<int32_t>(q), -static_cast<int32_t>(M.m))) + u;
                            part[ob][cb][r] |= res << sh;
                        }
            };
            if (M.divS == 0)
                epilogue(std::integral_constant<bool, false>{});
            else
                epilogue(std::integral_constant<bool, true>{});
        }
        // word w complete: store it.  Element (ob, cb, r) of this lane is
        // output channel og 64 + ob 16 + 4 (lane / 16) + r at position
        // x0 + cb 16 + lane % 16: a per-lane offset plus a uniform step.
        uint32_t *dstp = out + (static_cast<uint64_t>(M.woff) + w) * L.n_out + img * L.oN + row * L.oY +
                         x0 * L.oX + og * kLinOTile * L.oO;
        const uint32_t lo = 4 * (lane / 16) * L.oO + (lane % 16) * L.oX;
        if (full_tile) {
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        uint32_t *d = dstp + (ob * 16 + r) * L.oO + cb * 16 * L.oX;
                        d[lo] = part[ob][cb][r];
                        part[ob][cb][r] = 0;
                    }
        } else {
#pragma unroll
            for (int ob = 0; ob < 4; ++ob)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint32_t o = og * kLinOTile + o_local(ob, r), x = x0 + cb * 16 + lane % 16;
                        uint32_t *d = dstp + (ob * 16 + r) * L.oO + cb * 16 * L.oX;
                        if (o < L.c_out && x < L.cols) d[lo] = part[ob][cb][r];
                        part[ob][cb][r] = 0;
                    }
        }
    }
}

namespace {

int lin_launched() { return hipGetLastError() == hipSuccess ? REDASH_OK : REDASH_E_HIP; }

int lin_allow_lds(const void *kernel, uint32_t bytes) {
    if (bytes <= 64 * 1024) return REDASH_OK;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)) ==
                   hipSuccess
               ? REDASH_OK
               : REDASH_E_HIP;
}

template <int NCB, bool GARBLE, int K33, bool DEALT = false>
int launch_gemm(const LinPlan &L, const uint8_t *planes, const uint8_t *prep, const int64_t *bias,
                const uint32_t *offsets, uint32_t *out, hipStream_t stream) {
    int rc = lin_allow_lds(reinterpret_cast<const void *>(&k_linear_gemm<NCB, GARBLE, K33, DEALT>), L.lds_bytes);
    if (rc) return rc;
    const uint64_t tiles = static_cast<uint64_t>(L.nimg) * L.tile_rows * L.xtiles;
    if (tiles >= (1ull << 31)) return REDASH_E_PARAM;
    dim3 grid = L.word_split ? dim3(static_cast<uint32_t>(tiles), L.ogroups, L.npairs)
                             : dim3(static_cast<uint32_t>(tiles), L.k, L.ogroups);
    if constexpr (DEALT) {
        const uint64_t words = L.ogroups >= kXcds ? static_cast<uint64_t>(L.ogroups / kXcds) * L.npairs
                                                  : (L.npairs + kXcds / L.ogroups - 1) / (kXcds / L.ogroups);
        grid = dim3(static_cast<uint32_t>(kXcds * words * tiles));  // word_split: few
    }
    hipLaunchKernelGGL((k_linear_gemm<NCB, GARBLE, K33, DEALT>), grid, dim3(kLinBlock), L.lds_bytes, stream, L, planes,
                       prep, bias, offsets, out);
    return lin_launched();
}

template <int NCB, bool GARBLE, int K33>
int launch_gemm_w(const LinPlan &L, const uint8_t *planes, const uint8_t *prep, const int64_t *bias,
                  const uint32_t *offsets, uint32_t *out, hipStream_t stream) {
    constexpr int PL = K33 > 0 ? 7 : kWavePieces;
    if (L.kh * L.xw * (L.ck / 16) > 64u * PL || L.halo > 0xffffu) return REDASH_E_PARAM;  // not reached
    const uint32_t lds = L.lds_a + 4 * L.halo + 2 * kLinOTile * 4;
    int rc = lin_allow_lds(reinterpret_cast<const void *>(&k_linear_gemm_w<NCB, GARBLE, K33, PL>), lds);
    if (rc) return rc;
    const uint64_t tiles = static_cast<uint64_t>(L.nimg) * L.rows * L.xtiles;
    if (tiles >= (1ull << 31)) return REDASH_E_PARAM;
    const uint32_t nb = static_cast<uint32_t>((tiles + 3) / 4);
    hipLaunchKernelGGL((k_linear_gemm_w<NCB, GARBLE, K33, PL>),
                       L.word_split ? dim3(nb, L.ogroups, L.npairs) : dim3(nb, L.k, L.ogroups),
                       dim3(kLinBlock), lds, stream, L, planes, prep, bias, offsets, out);
    return lin_launched();
}

template <int NCB, bool GARBLE>
int launch_gemm_k(const LinPlan &L, const uint8_t *planes, const uint8_t *prep, const int64_t *bias,
                  const uint32_t *offsets, uint32_t *out, hipStream_t stream) {
    // one channel chunk (and a halo of at most 8 pieces per lane): independent waves
    if (L.ncc == 1 && L.kh * L.xw * (L.ck / 16) <= 64 * kWavePieces &&
        L.lds_a + 4 * L.halo + 2 * kLinOTile * 4 <= kLinMaxLds) {
        const bool k33 = L.kh == 3 && L.kw == 3 && L.ck == 64 && 3 * L.xw * 4 <= 7 * 64;
        if (k33 && L.xstride == 96) return launch_gemm_w<NCB, GARBLE, 96>(L, planes, prep, bias, offsets, out, stream);
        if (k33 && L.xstride == 80) return launch_gemm_w<NCB, GARBLE, 80>(L, planes, prep, bias, offsets, out, stream);
        return launch_gemm_w<NCB, GARBLE, 0>(L, planes, prep, bias, offsets, out, stream);
    }
    if (L.og_xcd)  // flattened: 3x3, stride 1
        return launch_gemm<NCB, GARBLE, 96, true>(L, planes, prep, bias, offsets, out, stream);
    if (L.kh == 3 && L.kw == 3 && L.ck == 64 && L.xstride == 96)
        return launch_gemm<NCB, GARBLE, 96>(L, planes, prep, bias, offsets, out, stream);
    if (L.kh == 3 && L.kw == 3 && L.ck == 64 && L.xstride == 80)
        return launch_gemm<NCB, GARBLE, 80>(L, planes, prep, bias, offsets, out, stream);
    return launch_gemm<NCB, GARBLE, 0>(L, planes, prep, bias, offsets, out, stream);
}

template <bool GARBLE>
int launch_linear(const LinPlan &L, const uint32_t *in, const uint8_t *prep, const int64_t *bias,
                  const uint32_t *offsets, uint8_t *work, uint32_t *out, hipStream_t stream) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return REDASH_E_HIP;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return REDASH_E_HIP;
    if (L.lds_bytes > static_cast<uint32_t>(v)) return REDASH_E_HIP;
    const uint64_t npos = static_cast<uint64_t>(L.nimg) * L.hp * L.wp;
    if (npos >= (1ull << 32)) return REDASH_E_PARAM;
    if (L.fold_c)
        hipLaunchKernelGGL(k_linear_unpack_rows, dim3(static_cast<uint32_t>((npos * L.cp + 1023) / 1024), L.npairs),
                           dim3(256), 0, stream, L, in, work);
    else
        hipLaunchKernelGGL(k_linear_unpack, dim3(static_cast<uint32_t>((npos + 63) / 64), L.npairs, (L.cp + 63) / 64),
                           dim3(256), 0, stream, L, in, work);
    if (lin_launched()) return REDASH_E_HIP;
    if (L.xt == 32) return launch_gemm_k<2, GARBLE>(L, work, prep, bias, offsets, out, stream);
    return launch_gemm_k<1, GARBLE>(L, work, prep, bias, offsets, out, stream);
}

}  // namespace

}  // namespace redash

using namespace redash;

extern "C" {

int redash_linear_plan(const redash_linear_params *p, redash_linear_sizes *out) {
    if (!p || !out) return REDASH_E_NULL;
    LinPlan L;
    const int rc = build_lin_plan(p, &L);
    if (rc) return rc;
    const uint32_t tw = total_words(L);
    out->in_label_words = L.n_in * tw;
    out->out_label_words = L.n_out * tw;
    out->prepared_bytes = prepared_bytes(L);
    out->work_bytes = work_bytes(L);
    out->h_out = (p->h_in + 2 * p->pad - p->kh) / p->stride + 1;
    out->w_out = (p->w_in + 2 * p->pad - p->kw) / p->stride + 1;
    out->offset_words = tw;
    return REDASH_OK;
}

int redash_linear_prepare(const redash_linear_params *p, const int32_t *d_weights, uint8_t *d_prepared,
                          hipStream_t stream) {
    LinPlan L;
    const int rc = build_lin_plan(p, &L);
    if (rc) return rc;
    if (!d_weights || !d_prepared) return REDASH_E_NULL;
    const uint64_t blocks = (L.rowsum_off + 255) / 256;
    hipLaunchKernelGGL(k_linear_prepare, dim3(static_cast<uint32_t>(blocks < 65536 ? blocks : 65536)), dim3(256),
                       0, stream, L, d_weights, d_prepared);
    if (lin_launched()) return REDASH_E_HIP;
    hipLaunchKernelGGL(k_linear_rowsums, dim3((L.k * L.o_pad + 255) / 256), dim3(256), 0, stream, L, d_weights,
                       d_prepared);
    return lin_launched();
}

int redash_linear_eval(const redash_linear_params *p, const uint32_t *d_in_labels, const uint8_t *d_prepared,
                       uint8_t *d_work, uint32_t *d_out_labels, hipStream_t stream) {
    LinPlan L;
    const int rc = build_lin_plan(p, &L);
    if (rc) return rc;
    if (!d_in_labels || !d_prepared || !d_work || !d_out_labels) return REDASH_E_NULL;
    return launch_linear<false>(L, d_in_labels, d_prepared, nullptr, nullptr, d_work, d_out_labels, stream);
}

int redash_linear_garble(const redash_linear_params *p, const uint32_t *d_in_zero, const uint8_t *d_prepared,
                         const int64_t *d_bias, const uint32_t *d_offsets, uint8_t *d_work, uint32_t *d_out_zero,
                         hipStream_t stream) {
    LinPlan L;
    const int rc = build_lin_plan(p, &L);
    if (rc) return rc;
    if (!d_in_zero || !d_prepared || !d_offsets || !d_work || !d_out_zero) return REDASH_E_NULL;
    return launch_linear<true>(L, d_in_zero, d_prepared, d_bias, d_offsets, d_work, d_out_zero, stream);
}

}  // extern "C"
