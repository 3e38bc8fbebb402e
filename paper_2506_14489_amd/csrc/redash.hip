// Kernels and C ABI of the ReDASH scaling-gadget library for gfx950.
//
// A large call evaluates one gadget per lane (k_eval); smaller ones spread a
// gadget's gates over waves (k_eval_split, k_garble) or over lanes
// (k_eval_small), encode and decode its moduli over workgroups and waves.
// Labels are packed words laid out [word][gadget], so a wavefront's label
// accesses are 64 consecutive words; the gate list and all per-modulus
// constants are uniform and come from the kernel argument block (scalar
// registers).  The AES round tables are staged into LDS once per workgroup.
// Nothing here uses MFMA: the work is table lookups, XORs, 32-bit multiplies
// for digit extraction and small modular arithmetic.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <mutex>

#include "../../include/redash.h"
#include "device.hpp"
#include "plan.hpp"

namespace redash {

struct SeedKey {
    uint32_t w[44];
};

// ---------------------------------------------------------------------------
// Evaluator: the hot path (Sec. 3.4 gadget, Sec. 2.3 projection gates).
//
// LDS of a workgroup (addresses from 0: the kernel declares no static LDS):
// the 64 KiB two-table image, the 88 round-key words, then one 128-byte
// free-operation table per gate (up to kMaxTables).  k_eval keeps a block's two
// target labels in registers from their first gate to their last; the other
// labels it reads are in global memory, mostly in L2 (the input, the output
// tensor, the working storage for Phase-B copies).  k_eval_split reads a gate's
// destination label and row there before the hash and writes the label back
// after it.  k_eval_small keeps every label of its gadgets in LDS, behind the
// tables.
// ---------------------------------------------------------------------------
constexpr uint32_t kEvalTableBase = kTableRegionBytes + 384;  // after the 352 key bytes
// LDS bytes of an evaluator workgroup with ntab free-operation tables.
constexpr uint32_t eval_lds_bytes(uint32_t ntab) { return kEvalTableBase + ntab * kTableBytes; }
static_assert(kLdsKeyWords * 4 <= 384, "round keys overlap the free-operation tables");
static_assert(2 * (kEvalTableBase + kMaxTables * kTableBytes) <= 160 * 1024, "two workgroups per CU");
static_assert(sizeof(EvalPlan) <= 4096, "the evaluator's plan is passed as its kernel argument block");
// The split evaluator: two workgroups of 768 threads share a CU (2 x 64.3 KiB
// of LDS), six waves per SIMD, which caps the kernel at 80 VGPRs.
constexpr int kEvalBlock = 768;
constexpr int kEvalWaves = 6;
// The one-gadget-per-lane evaluator k_eval: two workgroups of 1024, eight
// waves per SIMD at 64 VGPRs.  It is bound by the LDS pipe (25,800 table reads
// a wave, two cycles each) and the vector ALU together; what a wave waits for
// (reads of a round, rows) only other waves can fill, and eight waves with one
// gate hashed at a time beat six with two gates' blocks interleaved (80 VGPRs)
// and four on unrotated tables (128 KiB of them, 16 vector instructions fewer
// per round): 7.0, 7.5 and 8.0 ms at 3,211,264 gadgets of 77 gates.  A spill
// costs more than it moves: its reload waits for the row in flight.
constexpr int kLaneBlock = 1024;
constexpr int kLaneWaves = 8;
// The garbler: the same LDS image without the free-operation tables; two
// workgroups of 512 per CU, four waves per SIMD (92 VGPRs).  A gadget is a
// chain of 1,027 hashes on the 12-prime base, so calls that do not fill the
// chip split its gates over waves: 1,000 gadgets 6.98 -> 1.53 ms, 50,176
// 8.1 -> 3.0 ms; larger ones are bound by the vector ALU and the LDS pipe
// (200,704 gadgets 12.3 -> 10.0 ms, 802,816 42.2 -> 37.0 with shared rounds,
// truncated pads and rows subtracted a word at a time).
constexpr int kGarbleBlock = 512;
constexpr int kGarbleWaves = 4;

// The four places a label can be (kLocIn, kLocOut, kLocWork, kLocZero) for
// one thread: word w of a label starts at base + (offset + w) n, and the
// thread's gadget adds its byte offset 4 a (below 2^32).
struct LabelBufs {
    const uint32_t *in;
    uint32_t *out, *work;
    uint64_t n;
    uint32_t aoff;
    // word 0 of modulus mc's label in place `loc` (not kLocZero); uniform
    __device__ __forceinline__ const uint32_t *base(uint32_t loc, const ModConst &mc) const {
        if (loc == kLocIn) return in + static_cast<uint64_t>(mc.woff) * n;
        if (loc == kLocOut) return out + static_cast<uint64_t>(mc.woff) * n;
        return work + static_cast<uint64_t>(mc.wkoff) * n;
    }
    __device__ __forceinline__ uint32_t *dest(uint32_t to_work, const ModConst &mc) const {
        return to_work ? work + static_cast<uint64_t>(mc.wkoff) * n : out + static_cast<uint64_t>(mc.woff) * n;
    }
    // (opaque: the zero extension of the offset must sit next to the access,
    // or the scalar-base addressing form is not selected)
    __device__ __forceinline__ uint32_t get(const uint32_t *b, uint32_t w) const {
        return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(b + w * n) + opaque(aoff));
    }
    __device__ __forceinline__ void put(uint32_t *b, uint32_t w, uint32_t v) const {
        *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(b + w * n) + opaque(aoff)) = v;
    }
};

// A gate's free-operation table, four entries a lane: entry y is c' y mod m
// with c' = -c for a sub gate and c for an acc gate (fast_word).
__device__ __forceinline__ uint32_t free_op_entries(uint32_t lane, uint32_t kind, uint32_t c, uint32_t m) {
    const uint32_t cc = kind ? c : m - c;
    uint32_t w = 0;
    for (uint32_t k = 0; k < 4; ++k) w |= ((cc * (4 * lane + k)) % m) << (8 * k);
    return w;
}

// Fills the free-operation tables (gates 0..ntab-1 that have one).  Wave w
// fills gates w, w + waves, ...
__device__ __forceinline__ void stage_free_op_tables(const SplitPlan &P, uint32_t *lds, int tid, uint32_t nwaves) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(tid) / 64u);
    const uint32_t lane = static_cast<uint32_t>(tid) % 64u;
    for (uint32_t g = wave; g < P.ntab; g += nwaves) {
        const uint32_t d = P.gate[g];
        if (!gate_tab(d) || lane >= kTableBytes / 4) continue;
        lds[(kEvalTableBase + g * kTableBytes) / 4 + lane] =
            free_op_entries(lane, gate_kind(d), gate_coeff(d), P.mod[gate_dst(d)].m);
    }
}

// ---------------------------------------------------------------------------
// The one-gadget-per-lane evaluator, target-major (EvalPlan): a block's two
// target labels stay in registers from their first gate to their last, so
// each is read and written once; a step folds one digit label for one gate
// of each slot or for one slot, and takes its gates in turn.  Updates always
// act on slot 0: slot 1 is brought there by swapping the two slots.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void swap_slots(uint32_t (&T)[2][kMaxW]) {
    static_for<kMaxW>([&](auto w) {
        const uint32_t v = T[0][w];
        T[0][w] = T[1][w];
        T[1][w] = v;
    });
}

// Register labels are right-aligned: a label of W words sits in positions
// kMaxW - W .. kMaxW - 1 of its array (W is 4, 5 or 6), so its last word --
// the one with its own digit count -- is always at position kMaxW - 1 and
// every word is at a constant position: the word loops below are unrolled
// with a uniform test per position, and no register moves.
__device__ __forceinline__ uint32_t label_off(const ModConst &mc) { return kMaxW - mc.W; }

__device__ __forceinline__ void load_label(uint32_t (&T)[kMaxW], const LabelBufs &LB, uint32_t loc, const ModConst &mc,
                                           bool from_input) {
    static_for<kMaxW>([&](auto p) { T[p] = 0; });
    if (from_input) {
        const uint32_t off = label_off(mc);
        const uint32_t *b = LB.base(loc, mc);
        static_for<kMaxW>([&](auto p) {
            if (p >= static_cast<int>(off)) T[p] = LB.get(b, p - off);
        });
    }
}

__device__ __forceinline__ void store_label(const uint32_t (&T)[kMaxW], const LabelBufs &LB, uint32_t to_work,
                                            const ModConst &mc) {
    const uint32_t off = label_off(mc);
    uint32_t *b = LB.dest(to_work, mc);
    static_for<kMaxW>([&](auto p) {
        if (p >= static_cast<int>(off)) LB.put(b, p - off, T[p]);
    });
}

// A row of W words (4, 5 or 6, word-aligned), right-aligned like the labels:
// its last four words in one load.
__device__ __forceinline__ void load_row(uint32_t (&row)[kMaxW], const uint32_t *__restrict__ rp, uint32_t W) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
    const u4 v = *reinterpret_cast<const u4 *>(rp + (W - 4));
    row[2] = v.x;
    row[3] = v.y;
    row[4] = v.z;
    row[5] = v.w;
    if (W > 4) row[1] = rp[W - 5];
    if (W > 5) row[0] = rp[0];
}

// XOR-fold of a right-aligned register label with OFF = kMaxW - W: word w
// goes into lane w mod 4.
template <int OFF>
__device__ __forceinline__ void fold_regs(const uint32_t (&T)[kMaxW], uint32_t (&x)[4]) {
    static_for<kMaxW - OFF>([&](auto w) { x[w & 3] ^= T[w + OFF]; });
}

// Moduli without the fast constants (4 and 16, whose fields fill a word, and
// the primes 41, 47, 53, 59 and 61, whose split parts are too large for the
// 24-bit digit steps): one residue at a time with 32-bit divisions, over all
// kMaxW positions in a rolled loop that rotates the label, the row and the pad
// by one word per position (kMaxW rotations put label and row back in place).  The gadget
// configurations in use all take the fast path.
__device__ __forceinline__ void reg_update_generic(uint32_t e, const ModConst &mm, uint32_t (&Dw)[kMaxW],
                                                   uint32_t (&row)[kMaxW], uint32_t (&T)[kMaxW]) {
    const uint32_t coeff = eg_coeff(e), off = label_off(mm);
#pragma unroll 1
    for (uint32_t p = 0; p < static_cast<uint32_t>(kMaxW); ++p) {
        const uint32_t l = next_word(T);
        const uint32_t rw = next_word(row);
        uint32_t D = next_word(Dw);
        uint32_t res = l;
        if (p >= off) {
            const bool last = (p + 1 == static_cast<uint32_t>(kMaxW));
            const uint32_t nres = last ? mm.glast : mm.g;
            res = 0;
            for (uint32_t j = nres; j-- > 0;) {
                uint32_t pd;
                if (j) {
                    const uint32_t qd = div_m(D, mm);
                    pd = D - qd * mm.m;
                    D = qd;
                } else {
                    pd = D;
                }
                const uint32_t ev = add_mod(pd, field(rw, j, mm), mm.m);
                const uint32_t lj = field(l, j, mm);
                const uint32_t r = eg_kind(e) == 0 ? mul_mod(coeff, sub_mod(lj, ev, mm.m), mm)
                                                   : add_mod(lj, mul_mod(coeff, ev, mm), mm.m);
                res |= r << (mm.b * j);
            }
        }
        T[kMaxW - 1] = res;
        row[kMaxW - 1] = rw;
    }
}

// The full words (positions kMaxW - W .. kMaxW - 2) with the word shape
// (residues per word, bits per residue) known at compile time: the shape is
// dispatched once per gate, not once per word.  D[p] becomes the word's
// result (fast_word_c).
template <bool TAB, int NR, int BB>
__device__ __forceinline__ void reg_full_words(const ModConst &mm, uint32_t cc, uint32_t (&D)[kMaxW],
                                               const uint32_t (&row)[kMaxW], const uint32_t (&T)[kMaxW], uint32_t lmask,
                                               uint32_t km, uint64_t tk) {
    const uint32_t off = label_off(mm);
    static_for<kMaxW - 1>([&](auto p) {
        if (p > 0 || off == 0) {  // five or six words (fill_mod_const)
            D[p] = fast_word_c<NR, BB, TAB>(D[p], mm.lo_M_f, mm.lo_s_f, mm.pw_lo_f, mm.fc_hi_f, mm.fc_lo_f, row[p],
                                            T[p], lmask, km, cc, mm, tk);
        }
    });
}

template <bool TAB>
__device__ __forceinline__ void reg_update_fast(uint32_t e, const ModConst &mm, uint32_t (&D)[kMaxW],
                                                const uint32_t (&row)[kMaxW], uint32_t (&T)[kMaxW], uint64_t tk) {
    const bool acc = eg_kind(e) != 0;
    const uint32_t cc = acc ? eg_coeff(e) : mm.m - eg_coeff(e);  // c' (the coefficient is in 1..m-1)
    const uint32_t lmask = opaque(acc ? 0u : 0xffffffffu), km = opaque(acc ? 0u : mm.sw_ones * mm.m);
    // full words: g = floor(32 / b) residues of b bits
    switch (mm.fd ? mm.g | (mm.b << 8) : 0u) {
#define REDASH_FULL(NR, BB) \
    case (NR) | ((BB) << 8): reg_full_words<TAB, NR, BB>(mm, cc, D, row, T, lmask, km, tk); break;
        REDASH_FULL(16, 2) REDASH_FULL(10, 3) REDASH_FULL(8, 4) REDASH_FULL(6, 5) REDASH_FULL(5, 6)
        REDASH_FULL(4, 7) REDASH_FULL(4, 8)
#undef REDASH_FULL
        default: {
            const uint32_t off = label_off(mm);
            static_for<kMaxW - 1>([&](auto p) {
                if (p >= static_cast<int>(off)) {
                    D[p] = fast_word(D[p], mm.g, mm.nlo_f, mm.lo_M_f, mm.lo_s_f, mm.pw_lo_f, row[p], T[p], acc, cc, mm);
                }
            });
        }
    }
    D[kMaxW - 1] = fast_word_any<TAB>(D[kMaxW - 1], mm.glast, mm.nlo_l, mm.lo_M_l, mm.lo_s_l, mm.pw_lo_l, mm.fc_hi_l,
                                      mm.fc_lo_l, row[kMaxW - 1], T[kMaxW - 1], lmask, km, acc, cc, mm, tk);
    if (acc) {
        const uint32_t E = opaque(mm.sw_even);
        static_for<kMaxW>([&](auto p) { T[p] = swar_add(T[p], D[p] & E, (D[p] >> mm.b) & E, mm); });
    } else {
        static_for<kMaxW>([&](auto p) { T[p] = D[p]; });
    }
}

// Applies gate g's free operation to the register label T: E = row + pad,
// then L <- c (L - E) (sub: division step and the recursion of Eq.
// rns_to_mrs) or L <- L + c E (acc: the mixed-radix recombination onto a
// scaling modulus).  For an output modulus m <= 42 the products c' y mod m
// (fast_word) come from the gate's byte table in LDS.
// D: the gate's pad (pad_words_top, pad_words_all).
__device__ __forceinline__ void reg_update(uint32_t g, uint32_t e, const ModConst &mm, uint32_t (&D)[kMaxW],
                                           uint32_t (&row)[kMaxW], uint32_t (&T)[kMaxW]) {
    if (mm.m == 2) {  // W = 4: positions 2..5
        const bool flip = eg_kind(e) == 0 || (eg_coeff(e) & 1u);  // sub: q^{-1} = 1 mod 2
        if (flip) {
            static_for<4>([&](auto w) { T[w + 2] ^= D[w + 2] ^ row[w + 2]; });
        }
    } else if (eg_tab(e)) {
        reg_update_fast<true>(e, mm, D, row, T, opaque64(static_cast<uint64_t>(kEvalTableBase + g * kTableBytes) << 32));
    } else if (mm.fast) {
        reg_update_fast<false>(e, mm, D, row, T, 0);
    } else {
        reg_update_generic(e, mm, D, row, T);
    }
}

// The free-operation tables of an EvalPlan (as stage_free_op_tables).
__device__ __forceinline__ void stage_free_op_tables_e(const EvalPlan &P, uint32_t *lds, int tid, uint32_t nwaves) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(tid) / 64u);
    const uint32_t lane = static_cast<uint32_t>(tid) % 64u;
    for (uint32_t g = wave; g < P.ntab; g += nwaves) {
        const uint32_t e = P.egate[g];
        if (!eg_tab(e) || lane >= kTableBytes / 4) continue;
        lds[(kEvalTableBase + g * kTableBytes) / 4 + lane] =
            free_op_entries(lane, eg_kind(e), eg_coeff(e), P.mod[eg_dst(e)].m);
    }
}

// Gate g's pad from its hash fraction V: from the leading limbs (V[0..2] need
// not be there), or from all of them when the modulus takes all.  Where some
// lane's digits could depend on limbs 0-2 (about once in 2^12 waves) the
// wave hashes the gate's first block again for them: digit(x) reads and folds
// the digit label, tau() is the tweak.
template <typename Digit, typename Tau>
__device__ __forceinline__ void gate_pad(const PermTE02 &TT, const uint32_t *K, uint32_t gid, const ModConst &mm,
                                         uint32_t (&V)[8], uint32_t (&D)[kMaxW], Digit &&digit, Tau &&tau) {
    if (mm.pad_amb != 0) {
        const uint32_t v3 = V[3], v4 = V[4], v5 = V[5], v6 = V[6], v7 = V[7];
        if (__builtin_expect(!__any(pad_words_top(V, mm, D)), 1)) return;
        uint32_t x[4];
        digit(x);
        first_limbs(TT, LdsKey{K}, x, tau(), gid, V);
        V[3] = v3;
        V[4] = v4;
        V[5] = v5;
        V[6] = v6;
        V[7] = v7;
    }
    pad_words_all(V, mm, D);
}

// The gadget index a (below 2^30) is a 32-bit value: the row offset
// a (q-1) W + (c-1) W and the tweak (a0 + a) G + g are each 32 x 32 + 64-bit
// multiply-adds from it, instead of 64-bit values kept live across the gadget.
__device__ __forceinline__ uint64_t mad64(uint32_t x, uint32_t y, uint64_t z) {
    return static_cast<uint64_t>(x) * y + z;
}

// Gate g's tweak for local gadget a.
__device__ __forceinline__ uint64_t gate_tweak(const EvalPlan &P, uint32_t a, uint32_t g) {
    return mad64(a, P.G, P.a0 * P.G + g);
}

template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(kLaneWaves, kLaneWaves)))
k_eval(const EvalPlan P, const uint32_t *__restrict__ in, const uint32_t *__restrict__ tab, uint32_t *out,
       uint32_t *work) {
    extern __shared__ uint32_t lds[];
    uint32_t *K = lds + kTableRegionBytes / 4;
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;  // BLOCK or fewer (a multiple of 64)
    stage_perm_te02(lds, tid, nthr);
    stage_hash_key(K, tid, nthr);
    stage_free_op_tables_e(P, lds, tid, static_cast<uint32_t>(nthr) / 64u);
    __syncthreads();
    const PermTE02 TT = perm_te02();
    const uint32_t a0 = blockIdx.x * static_cast<uint32_t>(nthr) + static_cast<uint32_t>(tid);  // n < 2^30
    if (a0 >= P.n) return;  // no barrier follows
    // (only the byte offset 4 a stays in a register)
    const LabelBufs LB{in, out, work, P.n, opaque(a0 * 4u)};

    for (uint32_t b = 0; b < P.nblocks; ++b) {
        const uint32_t bd = P.block[b];
        uint32_t T[2][kMaxW];
        load_label(T[0], LB, kLocIn, P.mod[bk_mod0(bd)], bk_in0(bd) != 0);
        load_label(T[1], LB, kLocIn, P.mod[bk_mod1(bd)], bk_two(bd) && bk_in1(bd));
        const uint32_t s_end = bk_first(bd) + bk_steps(bd);
        for (uint32_t s = bk_first(bd); s < s_end; ++s) {
            const uint32_t sd = P.step[s];
            const bool two = st_two(sd) != 0;
            const bool alone1 = !two && st_slot1(sd);
            if (alone1) swap_slots(T);  // slot 1's gate acts on slot 0's registers
            // The digit label: folded into 128 bits for the hash, colour =
            // residue 0.  A residue >= q only occurs in a malformed input
            // label; it selects the implicit zero row, the output is garbage
            // and decode flags it.
            const ModConst mq = P.mod[st_dmod(sd)];
            const uint32_t q = mq.m;
            auto digit = [&](uint32_t(&x)[4]) -> uint32_t {
                static_for<4>([&](auto l) { x[l] = 0; });
                uint32_t w0, W = mq.W, loc = st_dloc(sd);
                // (kept here: for the rare second use nothing is computed ahead)
                asm volatile("" : "+s"(W), "+s"(loc));
                if (loc == kDigSlot0) {  // the block's first target, now in T[1]
                    switch (kMaxW - W) {
                        case 0: fold_regs<0>(T[1], x); w0 = T[1][0]; break;
                        case 1: fold_regs<1>(T[1], x); w0 = T[1][1]; break;
                        default: fold_regs<2>(T[1], x); w0 = T[1][2]; break;
                    }
                } else {
                    const uint32_t *dig = LB.base(loc, mq);
                    w0 = LB.get(dig, 0);
                    x[0] = w0;
                    static_for<kMaxW - 1>([&](auto w1) {
                        constexpr int w = decltype(w1)::value + 1;
                        if (w < static_cast<int>(W)) x[w & 3] ^= LB.get(dig, w);
                    });
                }
                return w0;
            };
            uint32_t x[4];
            const uint32_t w0 = digit(x);
            uint32_t colour = w0 & mq.mask;
            if (colour >= q) colour = 0;
            const uint32_t g = st_gate(sd);
            const uint32_t ng = two ? 2u : 1u;
#pragma unroll 1
            for (uint32_t j = 0; j < ng; ++j) {
                uint32_t e = P.egate[g + j];
                uint32_t row[kMaxW], V[8], D[kMaxW];
                static_for<kMaxW>([&](auto w) { row[w] = 0; });
                {
                    const uint32_t W = P.mod[eg_dst(e)].W;
                    if (colour != 0) {
                        // row (colour - 1) of the gadget's q - 1
                        const uint64_t at = static_cast<uint64_t>(eg_toff(e)) * P.n - W;
                        load_row(row, tab + mad64(opaque(colour), W, mad64(opaque(LB.aoff) >> 2, (q - 1) * W, at)), W);
                    }
                    hash_pair(TT, LdsKey{K}, x, [&] { return gate_tweak(P, opaque_here(LB.aoff) >> 2, g + j); }, P.gid,
                                  P.mod[eg_dst(e)].pad_amb == 0, V);
                }
                // (the modulus's constants are loaded here, not held in scalar
                // registers through the hash)
                asm volatile("" : "+s"(e));
                const ModConst mm = P.mod[eg_dst(e)];
                gate_pad(TT, K, P.gid, mm, V, D, digit, [&] { return gate_tweak(P, opaque(LB.aoff) >> 2, g + j); });
                reg_update(g + j, e, mm, D, row, T[0]);
                if (two) swap_slots(T);
            }
            if (alone1) swap_slots(T);
            const uint32_t f = st_store(sd);
            if (f & 3u) store_label(T[0], LB, (f >> 1) & 1u, P.mod[bk_mod0(bd)]);
            if ((f & 3u) == 3u) store_label(T[0], LB, 0, P.mod[bk_mod0(bd)]);
            if (f & 12u) store_label(T[1], LB, (f >> 3) & 1u, P.mod[bk_mod1(bd)]);
            if ((f & 12u) == 12u) store_label(T[1], LB, 0, P.mod[bk_mod1(bd)]);
        }
    }
}

// ---------------------------------------------------------------------------
// The evaluator for calls too small to fill the GPU one gadget per lane.
// A group of `split` waves shares 64 gadgets (one per lane); within a run of
// gates that share a digit label (distinct destinations, no dependence among
// them) wave j of the group takes gates j, j + split, ...; a workgroup
// barrier after each run makes the updated labels (in global memory; the
// waves of a workgroup share one write-through L1) visible to every wave
// before the next run reads them.  The gate a wave works on stays uniform.
// Same LDS image as k_eval.
//
// One launch may hold two kinds of workgroup: 0 .. nb0-1 give each group
// split0 waves, the others split1; the gadgets are first, first + 1, ... in
// workgroup order (blockDim / split0 per workgroup of the first kind, then
// blockDim / split1 per workgroup of the second).  The workgroups are
// dispatched in order, so the second kind takes the CUs the first frees.
// ---------------------------------------------------------------------------
struct SplitLaunch {
    uint32_t first;   // the launch's first gadget
    uint32_t nb0;     // workgroups of the first kind
    uint32_t split0;  // waves per 64 gadgets in them (2, 4 or 12)
    uint32_t split1;  // waves per 64 gadgets in the others
};
static_assert(sizeof(SplitPlan) + 4 * sizeof(void *) + sizeof(SplitLaunch) <= 4096,
              "the split evaluator's arguments fit the kernel argument block");

template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(kEvalWaves, kEvalWaves)))
k_eval_split(const SplitPlan P, const uint32_t *__restrict__ in, const uint32_t *__restrict__ tab, uint32_t *out,
             uint32_t *work, const SplitLaunch L) {
    extern __shared__ uint32_t lds[];
    uint32_t *K = lds + kTableRegionBytes / 4;
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;  // a multiple of 64 split0 and of 64 split1, at most BLOCK
    stage_perm_te02(lds, tid, nthr);
    stage_hash_key(K, tid, nthr);
    stage_free_op_tables(P, lds, tid, static_cast<uint32_t>(nthr) / 64u);
    __syncthreads();
    const PermTE02 TT = perm_te02();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(tid) / 64u);
    const uint32_t wg = blockIdx.x;
    const bool kind1 = wg >= L.nb0;
    const uint32_t split = kind1 ? L.split1 : L.split0;
    const uint32_t part = wave % split, grp = wave / split;
    const uint32_t per0 = static_cast<uint32_t>(nthr) / L.split0;
    const uint32_t start = kind1 ? L.nb0 * per0 + (wg - L.nb0) * (static_cast<uint32_t>(nthr) / L.split1) : wg * per0;
    const uint64_t a = static_cast<uint64_t>(L.first) + start + grp * 64u + static_cast<uint32_t>(tid) % 64u;
    const bool live = a < P.n;  // dead lanes still take every barrier
    const LabelBufs LB{in, out, work, P.n, static_cast<uint32_t>(live ? a : 0) * 4u};
    const uint64_t tau0 = (P.a0 + a) * P.G;
    for (uint32_t run = 0; run < P.nruns; ++run) {
        const uint32_t rd = P.run[run], g = rn_first(rd), r = rn_gates(rd);
        const ModConst mq = P.mod[rn_src(rd)];
        const uint32_t q = mq.m;
        // Every gate of the run hashes the same digit label: the wave reads,
        // folds and colours it once per run.
        uint32_t x[4] = {0, 0, 0, 0}, colour = 0;
        if (live && part < r) {
            const uint32_t *dig = LB.base(gate_dsrc(P.gate[g + part]), mq);
            const uint32_t w0 = LB.get(dig, 0);
            x[0] = w0;
            static_for<kMaxW - 1>([&](auto w1) {
                constexpr int w = decltype(w1)::value + 1;
                if (w < static_cast<int>(mq.W)) x[w & 3] ^= LB.get(dig, w);
            });
            colour = w0 & mq.mask;
            if (colour >= q) colour = 0;
        }
        for (uint32_t i = part; i < r; i += split) {
            if (!live) continue;  // (a lane's choice: the loop itself stays uniform)
            const uint32_t d = P.gate[g + i];
            const ModConst mm = P.mod[gate_dst(d)];
            const uint32_t Wd = mm.W;
            // the row (right-aligned, as the register labels)
            uint32_t row[kMaxW];
            static_for<kMaxW>([&](auto p) { row[p] = 0; });
            if (colour != 0)
                load_row(row, tab + static_cast<uint64_t>(P.goff[g + i]) * P.n + (a * (q - 1) + (colour - 1)) * Wd, Wd);
            uint32_t T[kMaxW];
            load_label(T, LB, gate_tsrc(d), mm, gate_tsrc(d) != kLocZero);
            uint32_t V[8], D[kMaxW];
            hash_pair(TT, LdsKey{K}, x, [&] { return opaque64(tau0 + g + i); }, P.gid, mm.pad_amb == 0, V);
            gate_pad(TT, K, P.gid, mm, V, D,
                     [&](uint32_t(&f)[4]) { static_for<4>([&](auto l) { f[l] = x[l]; }); },
                     [&] { return tau0 + g + i; });
            const uint32_t e = gate_dst(d) | (gate_kind(d) << 4) | (gate_tab(d) << 5) | (gate_coeff(d) << 6);
            reg_update(g + i, e, mm, D, row, T);
            store_label(T, LB, gate_tdst(d), mm);
        }
        __syncthreads();
    }
}

// The free operation of gate g (descriptor d) on one packed word of its label
// (reg_update for a single word w, which may differ between lanes): Dw the
// pad's digits of that word, rw the row's, l the label's.
__device__ __forceinline__ uint32_t word_update(uint32_t g, uint32_t d, const ModConst &mm, uint32_t Dw, uint32_t rw,
                                                uint32_t l, uint32_t w) {
    const bool acc = gate_kind(d) != 0;
    const uint32_t coeff = gate_coeff(d);
    if (mm.m == 2) return !acc || (coeff & 1u) ? l ^ Dw ^ rw : l;
    const bool last = w + 1 == mm.W;
    if (!mm.fast) {
        const uint32_t nres = last ? mm.glast : mm.g;
        uint32_t res = 0, D = Dw;
        for (uint32_t j = nres; j-- > 0;) {
            uint32_t pd = D;
            if (j) {
                const uint32_t qd = div_m(D, mm);
                pd = D - qd * mm.m;
                D = qd;
            }
            const uint32_t ev = add_mod(pd, field(rw, j, mm), mm.m), lj = field(l, j, mm);
            const uint32_t v = acc ? add_mod(lj, mul_mod(coeff, ev, mm), mm.m) : mul_mod(coeff, sub_mod(lj, ev, mm.m), mm);
            res |= v << (mm.b * j);
        }
        return res;
    }
    const uint32_t cc = acc ? coeff : mm.m - coeff;
    const uint32_t lmask = opaque(acc ? 0u : 0xffffffffu), km = opaque(acc ? 0u : mm.sw_ones * mm.m);
    const uint64_t tk = opaque64(static_cast<uint64_t>(kEvalTableBase + g * kTableBytes) << 32);
    uint32_t res = 0;
    // the full words' lanes, then the last word's (one copy of the shapes)
#pragma unroll 1
    for (uint32_t k = 0; k < 2; ++k) {
        const uint32_t nres = k ? mm.glast : mm.g, nlo = k ? mm.nlo_l : mm.nlo_f, lo_M = k ? mm.lo_M_l : mm.lo_M_f;
        const uint32_t lo_s = k ? mm.lo_s_l : mm.lo_s_f, pw_lo = k ? mm.pw_lo_l : mm.pw_lo_f;
        const uint32_t c_hi = k ? mm.fc_hi_l : mm.fc_hi_f, c_lo = k ? mm.fc_lo_l : mm.fc_lo_f;
        if (last == (k == 1)) {
            res = gate_tab(d) ? fast_word_any<true>(Dw, nres, nlo, lo_M, lo_s, pw_lo, c_hi, c_lo, rw, l, lmask, km, acc,
                                                    cc, mm, tk)
                              : fast_word_any<false>(Dw, nres, nlo, lo_M, lo_s, pw_lo, c_hi, c_lo, rw, l, lmask, km,
                                                     acc, cc, mm, 0);
        }
    }
    return acc ? swar_add(l, res & mm.sw_even, (res >> mm.b) & mm.sw_even, mm) : res;
}

// ---------------------------------------------------------------------------
// The evaluator for the smallest calls: at most kSmallMost gadgets per CU.
// A run of gates is two steps with a barrier after each.  Hash: a lane per
// (gate, gadget), so a wave's table reads serve 64 hashes where a wave per
// gate would serve as many as the workgroup has gadgets.  Update: a lane per
// (gadget, packed word), a wave (or two) per gate, whose modulus stays uniform;
// the full words and the last word take their shapes in two passes.  Every
// label of the workgroup's gadgets stays in LDS from the input to the output,
// and a run's rows are requested before its hashes.
// ---------------------------------------------------------------------------
// (12 primes, 77 gates: 1,000 gadgets 98 -> 66 us, 5,120 99 -> 79; one past,
// 84 us on the 12-wave split.)
constexpr uint32_t kSmallMost = 20;  // 6 words of 20 gadgets: two waves per gate
constexpr int kSmallTasks = 3;       // update waves per wave and run: 14 gates x 2 over 12 waves

struct SmallLaunch {
    uint32_t per;  // gadgets per workgroup, at most kSmallMost
};

// LDS words after the free-operation tables: the three label areas, then the
// hash fractions of a run's gates (8 limbs each).
__host__ __device__ constexpr uint32_t small_lds_words(uint32_t total_words, uint32_t work_words, uint32_t k,
                                                       uint32_t per) {
    return (2 * total_words + work_words) * per + 8 * k * per;
}

template <int BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_eval_small(const SplitPlan P, const uint32_t *__restrict__ in, const uint32_t *__restrict__ tab,
             uint32_t *__restrict__ out, const SmallLaunch L) {
    extern __shared__ uint32_t lds[];
    uint32_t *K = lds + kTableRegionBytes / 4;
    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / 64), c = L.per;
    uint32_t *lin = lds + (kEvalTableBase + P.ntab * kTableBytes) / 4;
    uint32_t *lout = lin + P.total_words * c, *lwork = lout + P.total_words * c, *Vb = lwork + P.work_words * c;
    const uint32_t a0 = blockIdx.x * c;  // the workgroup's first gadget
    const uint32_t nlive = P.n - a0 < c ? static_cast<uint32_t>(P.n - a0) : c;
    for (uint32_t e = tid; e < P.total_words * c; e += BLOCK) {
        const uint32_t w = e / c, gl = e % c;
        lin[e] = gl < nlive ? in[static_cast<uint64_t>(w) * P.n + a0 + gl] : 0u;
    }
    stage_perm_te02(lds, tid, BLOCK);
    stage_hash_key(K, tid, BLOCK);
    stage_free_op_tables(P, lds, tid, BLOCK / 64);
    const PermTE02 TT = perm_te02();
    // word 0 of modulus mc's labels in place `loc` (word w of gadget gl: [w c + gl])
    auto place = [&](uint32_t loc, const ModConst &mc) -> uint32_t * {
        return loc == kLocIn ? lin + mc.woff * c : loc == kLocOut ? lout + mc.woff * c : lwork + mc.wkoff * c;
    };
    for (uint32_t run = 0; run < P.nruns; ++run) {
        const uint32_t rd = P.run[run], g = rn_first(rd), r = rn_gates(rd), src = rn_src(rd), d0 = P.gate[g];
        const bool all = rn_all(rd) != 0;
        const uint32_t q = P.mod[src].m, Wq = P.mod[src].W, qmask = P.mod[src].mask;
        __syncthreads();  // the labels of the run before (or of the input) are in place
        const uint32_t *dig = place(gate_dsrc(d0), P.mod[src]);
        auto digit = [&](uint32_t gl, uint32_t(&x)[4]) {
            static_for<4>([&](auto l) { x[l] = 0; });
            static_for<kMaxW>([&](auto w) {
                if (w < static_cast<int>(Wq)) x[w & 3] ^= dig[w * c + gl];
            });
        };
        // The rows of this wave's update tasks: task t = wave, wave + 12, ...
        // is gate t / wpg of the run, its lane (t % wpg) 64 + lane the pair
        // (word, gadget).
        const uint32_t wpg = kMaxW * c > 64 ? 2u : 1u;
        uint32_t row[kSmallTasks];
        static_for<kSmallTasks>([&](auto u) {
            row[u] = 0;
            const uint32_t t = wave + u * (BLOCK / 64), i = t / wpg, idx = (t % wpg) * 64 + lane;
            if (i < r) {
                const uint32_t W = P.mod[gate_dst(P.gate[g + i])].W, w = idx / c, gl = idx % c;
                if (w < W && gl < nlive) {
                    uint32_t colour = dig[gl] & qmask;
                    if (colour >= q) colour = 0;
                    if (colour != 0)
                        row[u] = tab[static_cast<uint64_t>(P.goff[g + i]) * P.n +
                                     (static_cast<uint64_t>(a0 + gl) * (q - 1) + colour - 1) * W + w];
                }
            }
        });
        // Hashes: job i c + gl is gate g + i of gadget gl.
        if (wave * 64 < r * c) {
            const uint32_t job = tid < r * c ? tid : r * c - 1, i = job / c, gl = job % c;
            uint32_t x[4], V[8];
            digit(gl, x);
            hash_pair(TT, LdsKey{K}, x, [&] { return opaque64((P.a0 + a0 + gl) * P.G + g + i); }, P.gid, all, V);
            if (tid < r * c) static_for<8>([&](auto l) { Vb[l * (r * c) + job] = V[l]; });
        }
        __syncthreads();
        // Updates.
        static_for<kSmallTasks>([&](auto u) {
            const uint32_t t = wave + u * (BLOCK / 64), i = t / wpg, idx = (t % wpg) * 64 + lane;
            if (i < r) {
                const uint32_t d = P.gate[g + i];
                const ModConst mm = P.mod[gate_dst(d)];
                const uint32_t w = idx / c, gl = idx % c;
                if (w < mm.W) {
                    uint32_t V[8], D[kMaxW];
                    static_for<8>([&](auto l) { V[l] = Vb[l * (r * c) + i * c + gl]; });
                    gate_pad(TT, K, P.gid, mm, V, D, [&](uint32_t(&x)[4]) { digit(gl, x); },
                             [&] { return (P.a0 + a0 + gl) * P.G + g + i; });
                    const uint32_t at = w + label_off(mm);
                    uint32_t Dw = 0;
                    static_for<kMaxW>([&](auto p) { Dw = at == static_cast<uint32_t>(p) ? D[p] : Dw; });
                    uint32_t l = 0;
                    if (gate_tsrc(d) != kLocZero) l = place(gate_tsrc(d), mm)[w * c + gl];
                    place(gate_tdst(d) ? kLocWork : kLocOut, mm)[w * c + gl] = word_update(g + i, d, mm, Dw, row[u], l, w);
                }
            }
        });
    }
    __syncthreads();
    for (uint32_t e = tid; e < P.total_words * c; e += BLOCK) {
        const uint32_t w = e / c, gl = e % c;
        if (gl < nlive) out[static_cast<uint64_t>(w) * P.n + a0 + gl] = lout[e];
    }
}

// ---------------------------------------------------------------------------
// Garbler: offsets, zero-labels, garbled rows.
// ---------------------------------------------------------------------------

// Offsets R_m: digits of rho(1, i) in the radices (r0, m, m, ...), then
// residue 0 mapped to a unit of Z_m (d + 1 for a prime m, r0 = m - 1;
// 2d + 1 for m = 2^l, r0 = m/2), so that the m colours of a wire are
// distinct.  One thread per modulus.
__global__ void __launch_bounds__(64) k_offsets(const Plan P, const SeedKey key, uint32_t *__restrict__ offsets) {
    __shared__ uint32_t TT[kTableWords];
    stage_round_tables(TT, threadIdx.x, 64);
    __syncthreads();
    const uint32_t i = threadIdx.x;
    if (i >= P.k) return;
    const ModConst &mc = P.mod[i];
    uint32_t V[8];
    prg_fraction(TT, key.w, 1u, i, V);
    // residue 0, then the digits of a packed word at a time (the g - 1 left of
    // word 0, g of the next ones, glast of the last)
    const uint32_t d0 = frac_mul_carry(V, mc.r0);
    const uint32_t first = (mc.r0 == mc.m - 1) ? d0 + 1 : 2 * d0 + 1;
    for (uint32_t w = 0; w < mc.W; ++w) {
        const uint32_t nres = w + 1 == mc.W ? mc.glast : mc.g, j0 = w == 0 ? 1u : 0u;
        uint32_t pw = 1;  // m^(nres - j0); 0 stands for 2^32
        for (uint32_t j = j0; j < nres; ++j) pw *= mc.m;
        uint32_t D = nres > j0 ? frac_carry_any(V, pw) : 0u, word = w == 0 ? first : 0u;
        for (uint32_t j = nres; j-- > j0;) {
            const uint32_t q = D / mc.m;
            word |= (D - q * mc.m) << (mc.b * j);
            D = q;
        }
        offsets[mc.woff + w] = word;
    }
}

__device__ __forceinline__ uint32_t inverse_unit(uint32_t r, const ModConst &mc) {
    // r^(phi - 1) mod m for a unit r, phi the order of the unit group
    // (m - 1 for a prime, m/2 for a power of two)
    uint32_t e = mc.phi - 1, base = r, acc = 1 % mc.m;
    while (e) {
        if (e & 1u) acc = mul_mod(acc, base, mc);
        base = mul_mod(base, base, mc);
        e >>= 1;
    }
    return acc;
}

// The garbler's label access: like the evaluator's, except that a label read
// from the input tensor (the input zero-labels Z) is taken as Z - (P/2 mod m) R,
// the ShiftUp of Sec. 3.4 applied as a free constant addition.
// Right-aligned, as the register labels; its word 0 is at position `off`.
__device__ __forceinline__ void load_zero_label(const LabelBufs &LB, uint32_t loc, const ModConst &mc,
                                                const uint32_t *__restrict__ offsets, uint32_t (&L)[kMaxW]) {
    static_for<kMaxW>([&](auto p) { L[p] = 0; });
    if (loc == kLocZero) return;
    const uint32_t *b = LB.base(loc, mc);
    const uint32_t neg_up = (mc.m - mc.up) % mc.m;
    const int off = kMaxW - static_cast<int>(mc.W);
    static_for<kMaxW>([&](auto p) {
        if (p >= off) {
            L[p] = LB.get(b, p - off);
            if (loc == kLocIn) L[p] = label_axpy(L[p], offsets[mc.woff + p - off], neg_up, p - off, mc);
        }
    });
}

// A row of W words (4, 5 or 6) from a right-aligned register label.
__device__ __forceinline__ void store_row(const uint32_t (&row)[kMaxW], uint32_t *rp, uint32_t W) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
    u4 v;
    v.x = row[2];
    v.y = row[3];
    v.z = row[4];
    v.w = row[5];
    *reinterpret_cast<u4 *>(rp + (W - 4)) = v;
    if (W > 4) rp[W - 5] = row[1];
    if (W > 5) rp[0] = row[0];
}

// XOR-fold of a right-aligned label over the modulus mq.
__device__ __forceinline__ void fold_label(const uint32_t (&A)[kMaxW], const ModConst &mq, uint32_t (&x)[4]) {
    static_for<4>([&](auto l) { x[l] = 0; });
    switch (label_off(mq)) {
        case 0: fold_regs<0>(A, x); break;
        case 1: fold_regs<1>(A, x); break;
        default: fold_regs<2>(A, x); break;
    }
}

// Garbler (Sec. 2.3 projection gates with row reduction, the gadget of
// Sec. 3.4 applied to zero-labels).  `split` waves share 64 gadgets, one per
// lane: within a run of gates that share a digit label (distinct destinations)
// wave j of them takes gates j, j + split, ...; a workgroup barrier between
// runs publishes the updated labels.  Labels live where the evaluator keeps
// them (zin read with the ShiftUp, zout, work).
// Per gate q -> m the q labels of the digit wire are walked by colour:
// colour c holds the value v_c = (c - c_0) R_q[0]^{-1} mod q, so the label
// steps by the uniform label R_q[0]^{-1} R_q.  Colour 0 gives
// B0 = H(A_{v_0}) - (v_0 mod m) R_m; colour c >= 1 gives the row
// B0 + (v_c mod m) R_m - H(A_{v_c}).  The walk keeps B_c = B0 + (v_c mod m) R_m,
// starting from B_0 = H(A_{v_0}).
// GIVEN: the input zero-labels are the caller's (zin, read only; zin_w
// unused), e.g. the output zero-labels of a garbled linear layer; otherwise
// they are drawn from the PRG into zin_w (== zin).
template <int BLOCK, bool GIVEN>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(kGarbleWaves, kGarbleWaves)))
k_garble(const Plan P, const SeedKey key, const uint32_t *__restrict__ offsets, const uint32_t *zin,
         uint32_t *zin_w, uint32_t *zout, uint32_t *__restrict__ tab, uint32_t *work, uint32_t split) {
    extern __shared__ uint32_t lds[];
    uint32_t *K = lds + kTableRegionBytes / 4;
    const int tid = threadIdx.x;
    const int nthr = blockDim.x;  // BLOCK or fewer (a multiple of 64)
    stage_perm_te02(lds, tid, nthr);
    stage_hash_key(K, tid, nthr);
    __syncthreads();
    const PermTE02 TT = perm_te02();
    const LdsKey HK{K};
    const uint32_t wave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(tid) / 64u);
    const uint32_t part = wave % split;
    const uint64_t a = (static_cast<uint64_t>(blockIdx.x) * (static_cast<uint32_t>(nthr) / 64u / split) + wave / split) * 64u +
                       static_cast<uint32_t>(tid) % 64u;
    const bool live = a < P.n;  // dead lanes still take every barrier
    const uint64_t n = P.n;
    const uint64_t ga = P.a0 + a;
    const LabelBufs LB{zin, zout, work, n, static_cast<uint32_t>(live ? a : 0) * 4u};

    // Input zero-labels Z: digits of rho(2, ga k + i) (Sec. 2.3 label sampling).
    for (uint32_t i = part; i < (GIVEN || !live ? 0u : P.k); i += split) {
        const ModConst mc = P.mod[i];
        uint32_t s[1][4];
        uint32_t V[8];
        static_for<2>([&](auto h) {
            const uint64_t c = (ga * P.k + i) * 2u + static_cast<uint64_t>(h);
            s[0][0] = static_cast<uint32_t>(c);
            s[0][1] = static_cast<uint32_t>(c >> 32);
            s[0][2] = 0;
            s[0][3] = 2u << 24;
            aes128_encrypt_n<1>(TT, s, ArgKey{key.w});
            static_for<4>([&](auto l) { V[4 * h + l] = s[0][l]; });
        });
        uint32_t *dst = zin_w + static_cast<uint64_t>(mc.woff) * n;
        for (uint32_t w = 0; w < mc.W; ++w) LB.put(dst, w, prg_word(V, w, mc));
    }
    __syncthreads();

    const uint64_t tau0 = ga * P.G;
    uint64_t toff = 0;
    uint32_t run = 0;  // the first gate of the run of gates that share g's digit
    for (uint32_t g = 0; g < P.G; ++g) {
        const uint32_t d = P.gate[g];
        const ModConst mq = P.mod[gate_src(d)];
        const ModConst mm = P.mod[gate_dst(d)];
        if (g > 0 && gate_src(d) != gate_src(P.gate[g - 1])) {
            // the labels that the run before wrote are read from here on
            __syncthreads();
            run = g;
        }
        if ((g - run) % split != part || !live) {
            toff += n * (mq.m - 1) * mm.W;
            continue;
        }
        const uint32_t q = mq.m, m = mm.m;
        // (labels over the output modulus are right-aligned, as the pads)
        const int off = kMaxW - static_cast<int>(mm.W);
        uint32_t Rq[kMaxW], Rm[kMaxW];
        const int qoff = kMaxW - static_cast<int>(mq.W);
        static_for<kMaxW>([&](auto w) {
            Rq[w] = w >= qoff ? offsets[mq.woff + w - qoff] : 0u;
            Rm[w] = w >= off ? offsets[mm.woff + w - off] : 0u;
        });
        uint32_t A[kMaxW];
        load_zero_label(LB, gate_dsrc(d), mq, offsets, A);
        const uint32_t rinv = inverse_unit(offsets[mq.woff] & mq.mask, mq);
        // v: the value of colour 0; A <- A0 + v R_q
        const uint32_t a00 = (qoff == 0 ? A[0] : qoff == 1 ? A[1] : A[2]) & mq.mask;
        uint32_t v = mul_mod((q - a00) % q, rinv, mq);
        static_for<kMaxW>([&](auto w) {
            if (w >= qoff) A[w] = label_axpy(A[w], Rq[w], v, w - qoff, mq);
        });
        // uniform steps: the input label by rinv R_q, the output label by
        // (rinv mod m) R_m, or ((rinv - q) mod m) R_m when v wraps past q (in
        // vector registers: there are too many for the scalar ones)
        const uint32_t s1 = rinv % m, s2 = (rinv % m + m - q % m) % m;
        uint32_t Rse[kMaxW], Rso[kMaxW], U1[kMaxW], U2[kMaxW];
        static_for<kMaxW>([&](auto w) {
            const uint32_t rs = w >= qoff ? label_axpy(0u, Rq[w], rinv, w - qoff, mq) : 0u;
            Rse[w] = opaque(q == 2 ? rs : rs & mq.sw_even);
            Rso[w] = opaque((rs >> mq.b) & mq.sw_even);
            U1[w] = opaque(w >= off ? label_axpy(0u, Rm[w], s1, w - off, mm) : 0u);
            U2[w] = opaque(w >= off ? label_axpy(0u, Rm[w], s2, w - off, mm) : 0u);
        });
        uint32_t B[kMaxW];
        static_for<kMaxW>([&](auto w) { B[w] = 0; });
        uint32_t *row_at = tab + toff + a * (q - 1) * mm.W;
#pragma unroll 1
        for (uint32_t c = 0; c < q; ++c) {
            // (the moduli's constants are loaded where they are used, not held in
            // scalar registers through the hash: two sets do not fit)
            uint32_t dc = d;
            asm volatile("" : "+s"(dc));
            if (c != 0) {
                const ModConst mq = P.mod[gate_src(dc)], mm = P.mod[gate_dst(dc)];
                static_for<kMaxW>([&](auto w) {
                    if (w >= kMaxW - static_cast<int>(mq.W))
                        A[w] = q == 2 ? A[w] ^ Rse[w] : swar_add(A[w], Rse[w], Rso[w], mq);
                });
                const uint32_t vn = v + rinv;
                const bool wrap = vn >= q;
                v = wrap ? vn - q : vn;
                static_for<kMaxW>([&](auto w) {
                    if (w >= off) {
                        const uint32_t u = wrap ? U2[w] : U1[w];
                        B[w] = m == 2 ? B[w] ^ u : swar_add(B[w], u & mm.sw_even, (u >> mm.b) & mm.sw_even, mm);
                    }
                });
            }
            // the packed pad of the label A under the gate's tweak
            uint32_t x[4], V[8], D[kMaxW];
            fold_label(A, P.mod[gate_src(dc)], x);
            auto tweak = [&] { return opaque64(tau0 + g); };
            hash_pair(TT, HK, x, tweak, P.gid, P.mod[gate_dst(dc)].pad_amb == 0, V);
            asm volatile("" : "+s"(dc));
            const ModConst mm = P.mod[gate_dst(dc)];
            gate_pad(TT, K, P.gid, mm, V, D, [&](uint32_t(&f)[4]) { fold_label(A, P.mod[gate_src(dc)], f); }, tweak);
            pack_pad(D, mm);
            if (c != 0) {
                // colours 1..q-1: the row B_c - H(A_{v_c})
                static_for<kMaxW>([&](auto p) { D[p] = m == 2 ? B[p] ^ D[p] : swar_sub(B[p], D[p], mm.sw_ones * m, mm); });
                store_row(D, row_at, mm.W);
                row_at += mm.W;
            } else {
                // colour 0: the pad H(A_v0) starts the walk B_c = B0 + (v_c mod m) R_m,
                // with B0 = H(A_v0) - (v0 mod m) R_m (row reduction: no row stored);
                // the free operation on the destination zero-label is the
                // evaluator's on labels, E replaced by B0
                uint32_t T[kMaxW];
                load_zero_label(LB, gate_tsrc(d), mm, offsets, T);
                const uint32_t coeff = gate_coeff(d);
                const uint32_t negv = (m - v % m) % m;
                uint32_t *dst = LB.dest(gate_tdst(d), mm);
                static_for<kMaxW>([&](auto p) {
                    B[p] = D[p];
                    if (p >= off) {
                        const uint32_t w = p - off;
                        const uint32_t b0 = label_axpy(D[p], offsets[mm.woff + w], negv, w, mm);
                        LB.put(dst, w, gate_kind(d) == 0 ? label_scaled_sub(T[p], b0, coeff, w, mm)
                                                         : label_axpy(T[p], b0, coeff, w, mm));
                    }
                });
            }
        }
        toff += n * (q - 1) * mm.W;
    }
    // Output zero-labels: the working labels plus (P/(2s) mod m) R, the
    // ShiftDown of Sec. 3.4.
    __syncthreads();
    for (uint32_t i = live ? part : P.k; i < P.k; i += split) {
        const ModConst mc = P.mod[i];
        uint32_t *p = zout + static_cast<uint64_t>(mc.woff) * n;
        for (uint32_t w = 0; w < mc.W; ++w)
            LB.put(p, w, label_axpy(LB.get(p, w), offsets[mc.woff + w], mc.down, w, mc));
    }
}

// ---------------------------------------------------------------------------
// Encode (stand-in for oblivious transfer) and decode.
// ---------------------------------------------------------------------------
// x mod m of a signed 64-bit x: (hi 2^32 + lo) mod m by halves, 2^64 mod m
// taken off for a negative x.
__device__ __forceinline__ uint32_t mod64(int64_t x, uint32_t m) {
    const uint32_t lo = static_cast<uint32_t>(x), hi = static_cast<uint32_t>(static_cast<uint64_t>(x) >> 32);
    const uint32_t t = (0xffffffffu % m + 1u) % m;  // 2^32 mod m
    uint32_t r = ((hi % m) * t + lo % m) % m;       // below 2^16 + 2^8
    if (x < 0) r = (r + m * m - (t * t) % m) % m;   // 2^64 mod m = t^2 mod m
    return r;
}

// A workgroup takes 256 gadgets and PER moduli (blockIdx.y the group of them):
// the modulus is uniform, a small call still fills waves (65,536 gadgets over 10
// primes: 40 us with every modulus of a gadget on one lane, 14.5 with one per
// workgroup), and a large one streams whole kilobytes of each word.  P is a
// multiple of m_i: (x mod P) mod m_i = x mod m_i.
template <int BLOCK, uint32_t PER>
__global__ void __launch_bounds__(BLOCK) k_encode(const Plan P, const int64_t *__restrict__ x,
                                                  const uint32_t *__restrict__ zero,
                                                  const uint32_t *__restrict__ offsets, uint32_t *__restrict__ lab) {
    const uint64_t a = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x;
    if (a >= P.n) return;
    const uint64_t n = P.n;
    const int64_t xa = x[a];
#pragma unroll 1
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t i = blockIdx.y * PER + j;
        if (PER > 1 && i >= P.k) break;
        const ModConst mc = P.mod[i];
        const uint32_t v = mod64(xa, mc.m);
        const uint64_t base = static_cast<uint64_t>(mc.woff) * n + a;
        for (uint32_t w = 0; w < mc.W; ++w)
            lab[base + static_cast<uint64_t>(w) * n] =
                label_axpy(zero[base + static_cast<uint64_t>(w) * n], offsets[mc.woff + w], v, w, mc);
    }
}

__global__ void k_zero_u64(uint64_t *p) { *p = 0; }

// The CRT of the base: value = sum over i of (v_i c_i mod m_i) P / m_i, mod P,
// c_i = (P / m_i)^-1 mod m_i.
struct CrtConst {
    uint64_t quot[kMaxK];  // P / m_i
    uint32_t inv[kMaxK];   // c_i
};
static_assert(sizeof(Plan) + sizeof(CrtConst) + 6 * sizeof(void *) <= 4096, "decode's arguments fit the argument block");

// A workgroup takes 64 G gadgets with S waves per 64: wave (part, grp) checks
// the labels over moduli part, part + S, ... of group grp and finds their
// values; then the waves of part 0 sum the CRT terms of their gadgets (every
// partial sum reduced below P < 2^63) and count the bad ones.  G is at most 4
// (the terms in LDS), G S at most 16.
__global__ void __launch_bounds__(1024) k_decode(const Plan P, const CrtConst C, const uint32_t *__restrict__ Y,
                                                 const uint32_t *__restrict__ O, const uint32_t *__restrict__ offsets,
                                                 int64_t *__restrict__ y, unsigned long long *__restrict__ bad,
                                                 uint32_t G, uint32_t S) {
    __shared__ uint32_t terms[kMaxK * 256];  // v_i c_i mod m_i, bit 31: the label is not O + v R
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const uint32_t grp = wave % G, part = wave / G;
    uint32_t *term = terms + grp * (kMaxK * 64);
    const uint64_t a = (static_cast<uint64_t>(blockIdx.x) * G + grp) * 64 + lane;
    const uint64_t n = P.n;
    for (uint32_t i = part; i < P.k; i += S) {
        if (a >= n) continue;  // (a lane's choice: the loop itself stays uniform)
        const ModConst mc = P.mod[i];
        const uint64_t base = static_cast<uint64_t>(mc.woff) * n + a;
        const uint32_t y0 = Y[base] & mc.mask, o0 = O[base] & mc.mask;
        const uint32_t vi = mul_mod(sub_mod(y0, o0, mc.m), inverse_unit(offsets[mc.woff] & mc.mask, mc), mc);
        bool ok = true;
        for (uint32_t w = 0; w < mc.W; ++w) {
            const uint64_t at = base + static_cast<uint64_t>(w) * n;
            if (label_axpy(O[at], offsets[mc.woff + w], vi, w, mc) != Y[at]) ok = false;
        }
        // (a malformed label's value may be m or more: reduced for the sum)
        term[i * 64 + lane] = ((vi % mc.m) * C.inv[i]) % mc.m | (ok ? 0u : 0x80000000u);
    }
    __syncthreads();
    if (part != 0 || a >= n) return;
    uint64_t val = 0;
    uint32_t flags = 0;
    for (uint32_t j = 0; j < P.k; ++j) {
        const uint32_t t = term[j * 64 + lane];
        flags |= t;
        val += static_cast<uint64_t>(t & 0xffu) * C.quot[j];  // t P / m < P: the sum is below 2 P < 2^64
        if (val >= P.P) val -= P.P;
    }
    // signed range [-floor(P/2), ceil(P/2) - 1] (Sec. 2.4)
    int64_t out = static_cast<int64_t>(val);
    if (val >= (P.P + 1) / 2) out -= static_cast<int64_t>(P.P);
    y[a] = out;
    const uint64_t wrong = __ballot(flags >> 31);
    if (wrong && lane == static_cast<uint32_t>(__ffsll(static_cast<unsigned long long>(wrong)) - 1))
        atomicAdd(bad, static_cast<unsigned long long>(__popcll(wrong)));
}

// ---------------------------------------------------------------------------
// The hash alone.
// ---------------------------------------------------------------------------
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_hash(const ModConst mq, const ModConst mm, uint64_t count,
                                                const uint32_t *__restrict__ lab, uint32_t gid,
                                                const uint64_t *__restrict__ tau, uint32_t *__restrict__ out) {
    __shared__ uint32_t TT[kTableWords];
    stage_round_tables(TT, threadIdx.x, BLOCK);
    __syncthreads();
    const uint64_t a = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x;
    if (a >= count) return;
    uint32_t x[4] = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < kMaxW; ++w)
        if (w < static_cast<int>(mq.W)) x[w & 3] ^= lab[static_cast<uint64_t>(w) * count + a];
    uint32_t V[8];
    hash_fraction(TT, x[0], x[1], x[2], x[3], tau[a], gid, mm.m != 2, V);
#pragma unroll
    for (int w = 0; w < kMaxW; ++w)
        if (w < static_cast<int>(mm.W)) out[static_cast<uint64_t>(w) * count + a] = pad_word(V, w, mm);
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {

constexpr int kMaxDevices = 64;

// Per device: its compute units and the largest LDS allocation a block may
// request, read on the first call that runs on it (they do not change while
// the process runs).
struct DeviceInfo {
    int cus, max_lds;
};
std::mutex g_dev_mu;
DeviceInfo g_dev[kMaxDevices] = {};

int device_info(DeviceInfo *out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return REDASH_E_HIP;
    std::lock_guard<std::mutex> lock(g_dev_mu);
    DeviceInfo &d = g_dev[dev];
    if (d.cus <= 0) {
        int cus = 0, lds = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            return REDASH_E_HIP;
        if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
            return REDASH_E_HIP;
        d = DeviceInfo{cus, lds};
    }
    *out = d;
    return REDASH_OK;
}

// The plan of the parameters this host thread passed last, and its
// evaluator schedule once a call needed it: a layer evaluated call after call
// with the same parameters builds them once.  (redash_params has no padding:
// equal bytes are equal parameters; unused entries that differ only cost a
// rebuild.)
struct PlanCache {
    bool valid, has_eval, has_split;
    redash_params p;
    Plan P;
    EvalPlan E;
    SplitPlan S;
};
thread_local PlanCache t_plan;

int cached_plan(const redash_params *p, const Plan **out) {
    if (!p) return REDASH_E_NULL;
    PlanCache &c = t_plan;
    if (!c.valid || memcmp(&c.p, p, sizeof *p) != 0) {
        c.valid = false;
        const int rc = build_plan(p, &c.P);
        if (rc) return rc;
        c.p = *p;
        c.valid = true;
        c.has_eval = c.has_split = false;
    }
    *out = &c.P;
    return REDASH_OK;
}

// The evaluator schedule and the runs of the cached plan, which every entry
// point launches from (cached_plan), kept with it.
const EvalPlan &eval_plan() {
    PlanCache &c = t_plan;
    if (!c.has_eval) {
        build_eval_plan(c.P, &c.E);
        c.has_eval = true;
    }
    return c.E;
}

const SplitPlan &split_plan() {
    PlanCache &c = t_plan;
    if (!c.has_split) {
        build_split_plan(c.P, &c.S);
        c.has_split = true;
    }
    return c.S;
}

// Threads per workgroup for n gadgets: the smallest multiple of 64 that keeps
// the grid within one round of two workgroups per CU (the LDS image allows two),
// at most `most`.  Small launches thus spread over every CU instead of filling
// a few with long-running waves; large ones use `most`.
int block_for(uint64_t n, int most, int *out) {
    DeviceInfo d;
    const int rc = device_info(&d);
    if (rc) return rc;
    const uint64_t slots = 2ull * static_cast<uint64_t>(d.cus);
    const uint64_t b = 64 * ((n + 64 * slots - 1) / (64 * slots));
    *out = b < 64 ? 64 : (b > static_cast<uint64_t>(most) ? most : static_cast<int>(b));
    return REDASH_OK;
}

// Largest LDS allocation a block may request on the current device.
int max_lds_bytes(size_t *out) {
    DeviceInfo d;
    const int rc = device_info(&d);
    if (rc) return rc;
    *out = static_cast<size_t>(d.max_lds);
    return REDASH_OK;
}

// Allows a kernel to use more than the default 64 KiB of dynamic LDS.
int allow_lds(const void *kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return REDASH_OK;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)) ==
                   hipSuccess
               ? REDASH_OK
               : REDASH_E_HIP;
}

unsigned grid_for(uint64_t n, int block) { return static_cast<unsigned>((n + block - 1) / block); }

int launched() {
    return hipGetLastError() == hipSuccess ? REDASH_OK : REDASH_E_HIP;
}

// Launches k_eval_split (it may use more than 64 KiB of LDS).
int launch_split_kernel(const SplitPlan &P, uint32_t lds, const uint32_t *in, const uint32_t *tab, uint32_t *out,
                        uint32_t *work, const SplitLaunch &L, unsigned grid, int threads, hipStream_t stream) {
    const int rc = allow_lds(reinterpret_cast<const void *>(&k_eval_split<kEvalBlock>), lds);
    if (rc) return rc;
    hipLaunchKernelGGL(k_eval_split<kEvalBlock>, dim3(grid), dim3(threads), lds, stream, P, in, tab, out, work, L);
    return launched();
}

// Gadgets per workgroup of the split evaluator at full size: a multiple of 64
// with per * split <= kEvalBlock (768, 384, 192 and 64 for 1, 2, 4 and 12 waves).
constexpr uint32_t split_most(uint32_t split) { return kEvalBlock / split / 64 * 64; }

// k_eval_split over gadgets first .. first + count - 1 (of the plan's n), each
// group of 64 gadgets on `split` waves (12, 4 or 2).
int launch_split(uint32_t split, const SplitPlan &P, uint32_t lds, const uint32_t *in, const uint32_t *tab, uint32_t *out,
                 uint32_t *work, uint64_t first, uint64_t count, hipStream_t stream) {
    int per = 0;
    const int rc = block_for(count, static_cast<int>(split_most(split)), &per);
    if (rc) return rc;
    const SplitLaunch L{static_cast<uint32_t>(first), grid_for(count, per), split, split};
    return launch_split_kernel(P, lds, in, tab, out, work, L, grid_for(count, per), per * static_cast<int>(split),
                               stream);
}

// The split evaluator for `count` gadgets that one round of two workgroups
// per CU holds with 64, 192 or 384 gadgets per workgroup (12, 4 or 2 waves
// per 64 gadgets); 0 when the count needs more than one such round.
uint32_t split_for(uint64_t count, uint64_t cus) {
    if (count <= 2 * cus * 64) return 12;
    if (count <= 2 * cus * kEvalBlock / 4) return 4;
    if (count <= 2 * cus * kEvalBlock / 2) return 2;
    return 0;
}

// Launches the evaluators for n gadgets.  A call of at most kSmallMost gadgets
// per CU runs on k_eval_small.  A call that one round of two
// workgroups per CU holds when a gadget takes 12, 4 or 2 waves runs on
// k_eval_split with that split (runs of gates sharing a digit have at most
// k - 1 gates, 11 on the 12-prime base: with 12 waves one gate per wave and
// run).  A call a little above one full round of the 4- or 2-wave split
// (98,304 or 196,608 gadgets on 256 CUs, plus at most 64 gadgets per CU) runs
// that round and its rest as one launch, the rest's workgroups on 12 waves per
// 64 gadgets after the round's: they take the CUs the round frees first,
// instead of adding a wave to some SIMDs for the whole call.  A larger call
// runs on k_eval, one gadget per lane: whole rounds of two full workgroups per
// CU, and a rest that the 12- or 4-wave split holds in one round goes to it
// after them instead of running as a last round with few waves per SIMD, whose
// gadgets would take the latency of their gate chain (12 primes: 3,211,264
// gadgets, 65,536 over six rounds, 7.35 -> 7.00 ms; 622,592 1.57 -> 1.46; a
// rest of 175,712 costs the same either way).  Over rests of 8,192 to 98,304 after
// 1, 2, 3 and 6 rounds the split takes 0.88 to 1.02 of the time of k_eval for the
// rest with 14, 20, 27, 35, 54 and 77 gates (no base has 11 to 13), 0.91 to 1.07
// with 9 and 10 and 0.97 to 1.06 with 5, whose chains are short enough as they
// are: there only a rest of up to 32,768 goes to it.  A larger rest over one
// round makes two even rounds of smaller workgroups: a CU whose two workgroups
// end together would otherwise take two full ones of the rest and another CU
// none (802,816 gadgets 2.12 -> 1.90 ms).  Three even rounds take 0.94 to 1.07 of
// the time, as the rest falls (131,072 over two: 0.96, 200,000: 1.05, 300,000:
// 0.97), four or seven 1.00 to 1.08.
int launch_eval(const Plan &P, uint32_t lds, const uint32_t *in, const uint32_t *tab, uint32_t *out, uint32_t *work,
                hipStream_t stream) {
    DeviceInfo d;
    int rc = device_info(&d);
    if (rc) return rc;
    const uint64_t ncu = static_cast<uint64_t>(d.cus);
    if (P.n <= ncu * kSmallMost) {
        const uint32_t per = static_cast<uint32_t>((P.n + ncu - 1) / ncu);
        const uint32_t bytes = lds + 4 * small_lds_words(P.total_words, P.work_words, P.k, per);
        if (bytes <= static_cast<uint32_t>(d.max_lds)) {
            if ((rc = allow_lds(reinterpret_cast<const void *>(&k_eval_small<kEvalBlock>), bytes))) return rc;
            hipLaunchKernelGGL(k_eval_small<kEvalBlock>, dim3(grid_for(P.n, static_cast<int>(per))), dim3(kEvalBlock),
                               bytes, stream, split_plan(), in, tab, out, SmallLaunch{per});
            return launched();
        }
    }
    for (const uint32_t split : {4u, 2u}) {
        const uint32_t per0 = split_most(split);
        const uint64_t full = 2 * ncu * per0;
        if (P.n > full && P.n - full <= ncu * 64) {
            const uint32_t nb0 = static_cast<uint32_t>(2 * ncu);
            const unsigned grid = nb0 + grid_for(P.n - full, 64);
            return launch_split_kernel(split_plan(), lds, in, tab, out, work, SplitLaunch{0, nb0, split, 12}, grid, kEvalBlock,
                                       stream);
        }
    }
    if (const uint32_t split = split_for(P.n, ncu))
        return launch_split(split, split_plan(), lds, in, tab, out, work, 0, P.n, stream);
    const uint64_t round = 2 * ncu * kLaneBlock;  // gadgets of one round, one per lane
    uint64_t bulk = P.n;
    const uint64_t rest = P.n % round;
    if (P.n > round && rest > 0 && rest <= (P.G >= 14 ? 2 * ncu * split_most(4) : 2 * ncu * 64)) bulk = P.n - rest;
    if ((rc = allow_lds(reinterpret_cast<const void *>(&k_eval<kLaneBlock>), lds))) return rc;
    int block = 0;
    if ((rc = block_for(bulk > round && bulk < 2 * round ? (bulk + 1) / 2 : bulk, kLaneBlock, &block))) return rc;
    const EvalPlan &E = eval_plan();
    hipLaunchKernelGGL(k_eval<kLaneBlock>, dim3(grid_for(bulk, block)), dim3(block), lds, stream, E, in, tab, out,
                       work);
    if ((rc = launched())) return rc;
    if (bulk == P.n) return REDASH_OK;
    return launch_split(split_for(P.n - bulk, ncu), split_plan(), lds, in, tab, out, work, bulk, P.n - bulk, stream);
}


SeedKey seed_key(uint64_t seed) {
    RoundKeys rk = make_seed_round_keys(seed);
    SeedKey k;
    memcpy(k.w, rk.w, sizeof k.w);
    return k;
}

}  // namespace

}  // namespace redash

using namespace redash;

extern "C" {

int redash_plan(const redash_params *p, redash_sizes *out) {
    if (!p || !out) return REDASH_E_NULL;
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    out->label_words = P.n * P.total_words;
    uint64_t tw = 0;
    for (uint32_t g = 0; g < P.G; ++g) {
        const uint32_t d = P.gate[g];
        tw += P.n * (P.mod[gate_src(d)].m - 1) * P.mod[gate_dst(d)].W;
    }
    out->table_words = tw;
    out->offset_words = P.total_words;
    out->gates = P.G;
    out->work_words = P.n * P.work_words;
    return REDASH_OK;
}

}  // extern "C"

namespace {

template <bool GIVEN>
int garble_scale(const redash_params *p, uint32_t *d_offsets, const uint32_t *d_in_zero, uint32_t *d_in_zero_w,
                 uint32_t *d_out_zero, uint32_t *d_tables, uint32_t *d_work, hipStream_t stream) {
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    if (P.n >= (1ull << 30)) return REDASH_E_PARAM;  // 4 a must fit in 32 bits
    if (!d_offsets) return REDASH_E_NULL;
    if (P.n > 0 && (!d_in_zero || !d_out_zero || !d_tables || (P.work_words && !d_work))) return REDASH_E_NULL;
    const SeedKey key = seed_key(P.seed);
    hipLaunchKernelGGL(k_offsets, dim3(1), dim3(64), 0, stream, P, key, d_offsets);
    if ((rc = launched())) return rc;
    if (P.n == 0) return REDASH_OK;
    size_t max_lds = 0;
    if ((rc = max_lds_bytes(&max_lds))) return rc;
    const uint32_t lds = kEvalTableBase;  // the AES image and the round keys
    if (lds > max_lds) return REDASH_E_HIP;
    if ((rc = allow_lds(reinterpret_cast<const void *>(&k_garble<kGarbleBlock, GIVEN>), lds))) return rc;
    // waves per 64 gadgets: as many as one round of two workgroups per CU
    // holds (a gadget's gates in turn are a long chain), at most 8
    DeviceInfo dev;
    if ((rc = device_info(&dev))) return rc;
    uint32_t split = 8;
    while (split > 1 && P.n > 2ull * static_cast<uint64_t>(dev.cus) * (kGarbleBlock / split)) split /= 2;
    int per = 0;  // gadgets per workgroup
    if ((rc = block_for(P.n, kGarbleBlock / static_cast<int>(split), &per))) return rc;
    hipLaunchKernelGGL((k_garble<kGarbleBlock, GIVEN>), dim3(grid_for(P.n, per)), dim3(per * static_cast<int>(split)), lds,
                       stream, P, key, d_offsets, d_in_zero, d_in_zero_w, d_out_zero, d_tables, d_work, split);
    return launched();
}

}  // namespace

extern "C" {

int redash_garble_scale(const redash_params *p, uint32_t *d_offsets, uint32_t *d_in_zero, uint32_t *d_out_zero,
                        uint32_t *d_tables, uint32_t *d_work, hipStream_t stream) {
    return garble_scale<false>(p, d_offsets, d_in_zero, d_in_zero, d_out_zero, d_tables, d_work, stream);
}

int redash_garble_scale_given(const redash_params *p, uint32_t *d_offsets, const uint32_t *d_in_zero,
                              uint32_t *d_out_zero, uint32_t *d_tables, uint32_t *d_work, hipStream_t stream) {
    return garble_scale<true>(p, d_offsets, d_in_zero, nullptr, d_out_zero, d_tables, d_work, stream);
}

int redash_encode(const redash_params *p, const int64_t *d_x, const uint32_t *d_in_zero, const uint32_t *d_offsets,
                  uint32_t *d_in_labels, hipStream_t stream) {
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    if (!d_offsets) return REDASH_E_NULL;
    if (P.n == 0) return REDASH_OK;
    if (!d_x || !d_in_zero || !d_in_labels) return REDASH_E_NULL;
    // One modulus per workgroup while the call needs the workgroups; four, which
    // read the values once for all of them, where their workgroups (two groups of
    // moduli weigh as much as two moduli alone) pass 2^21 gadgets: 3,211,264
    // gadgets: 12 primes 633 -> 592 us, 5 primes 303 -> 292, 4 moduli 202 -> 191;
    // 800,000: 10 primes 142 -> 136; the other way at 1,100,000 with 3 and 4 moduli,
    // 37.0 -> 40.2 and 63.5 -> 69.1, and at 400,000 with 12 primes, 74 -> 79.
    const uint64_t groups = P.k == 2 ? 2 : (P.k + 3) / 4;
    if (P.n * groups > (1u << 21))
        hipLaunchKernelGGL((k_encode<256, 4>), dim3(grid_for(P.n, 256), (P.k + 3) / 4), dim3(256), 0, stream, P, d_x,
                           d_in_zero, d_offsets, d_in_labels);
    else
        hipLaunchKernelGGL((k_encode<256, 1>), dim3(grid_for(P.n, 256), P.k), dim3(256), 0, stream, P, d_x, d_in_zero,
                           d_offsets, d_in_labels);
    return launched();
}

int redash_eval_scale(const redash_params *p, const uint32_t *d_in_labels, const uint32_t *d_tables,
                      uint32_t *d_out_labels, uint32_t *d_work, hipStream_t stream) {
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    if (P.n >= (1ull << 30)) return REDASH_E_PARAM;  // 4 a must fit in 32 bits
    if (P.n == 0) return REDASH_OK;
    if (!d_in_labels || !d_tables || !d_out_labels || (P.work_words && !d_work)) return REDASH_E_NULL;
    size_t max_lds = 0;
    if ((rc = max_lds_bytes(&max_lds))) return rc;
    const uint32_t lds = eval_lds_bytes(P.ntab);
    if (lds > max_lds) return REDASH_E_HIP;
    return launch_eval(P, lds, d_in_labels, d_tables, d_out_labels, d_work, stream);
}

}  // extern "C"

namespace {

// Working storage of redash_eval_scale_noalloc.  In host code the name
// `scratch` only stands in for the device array: kernels get the device
// address that hipGetSymbolAddress returns on each GPU (every GPU holds its
// own copy at its own address).
__device__ __align__(256) uint32_t scratch[REDASH_NOALLOC_WORK_WORDS];

std::mutex g_scratch_mu;
uint32_t *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current GPU's scratch array, looked up once per GPU
// (with that GPU current) on its first use.
int scratch_address(uint32_t **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return REDASH_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return REDASH_E_HIP;
        g_scratch_ptr[dev] = static_cast<uint32_t *>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return REDASH_OK;
}

}  // namespace

extern "C" {

int redash_eval_scale_noalloc(const redash_params *p, const uint32_t *d_in_labels, const uint32_t *d_tables,
                              uint32_t *d_out_labels, hipStream_t stream) {
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    if (P.n >= (1ull << 30)) return REDASH_E_PARAM;  // 4 a must fit in 32 bits
    if (P.n * P.work_words > REDASH_NOALLOC_WORK_WORDS) return REDASH_E_SIZE;
    if (P.n == 0) return REDASH_OK;
    if (!d_in_labels || !d_tables || !d_out_labels) return REDASH_E_NULL;
    uint32_t *work = nullptr;
    if ((rc = scratch_address(&work))) return rc;
    size_t max_lds = 0;
    if ((rc = max_lds_bytes(&max_lds))) return rc;
    const uint32_t lds = eval_lds_bytes(P.ntab);
    if (lds > max_lds) return REDASH_E_HIP;
    return launch_eval(P, lds, d_in_labels, d_tables, d_out_labels, work, stream);
}

int redash_decode(const redash_params *p, const uint32_t *d_out_labels, const uint32_t *d_out_zero,
                  const uint32_t *d_offsets, int64_t *d_y, uint64_t *d_bad_count, hipStream_t stream) {
    const Plan *PP = nullptr;
    int rc = cached_plan(p, &PP);
    if (rc) return rc;
    const Plan &P = *PP;
    if (!d_offsets || !d_bad_count) return REDASH_E_NULL;
    if (P.n > 0 && (!d_out_labels || !d_out_zero || !d_y)) return REDASH_E_NULL;
    unsigned long long *bad = reinterpret_cast<unsigned long long *>(d_bad_count);
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(1), 0, stream, reinterpret_cast<uint64_t *>(bad));
    if ((rc = launched())) return rc;
    if (P.n == 0) return REDASH_OK;
    CrtConst C;
    memset(&C, 0, sizeof C);
    for (uint32_t i = 0; i < P.k; ++i) {
        C.quot[i] = P.P / P.mod[i].m;
        C.inv[i] = inverse_mod(static_cast<uint32_t>(C.quot[i] % P.mod[i].m), P.mod[i].m);
    }
    // Waves per 64 gadgets (S) and groups of 64 per workgroup (G).  A small
    // call takes a wave per modulus (12 primes, 65,536 gadgets: 69 us with every
    // modulus on one lane, 22), with two groups where that makes workgroups of
    // two waves (2 moduli, 262,144 gadgets: 21.6 us with one, 15.9).  A large one
    // has waves enough: fewer of them per group leave fewer idle, those past the
    // moduli or beside the one that sums.  From 4 moduli on S = 4 past 2^18 gadgets
    // (12 moduli at 262,144: 77.4 -> 65.2 us) and 2 past 2^19 (400,000, S = 4 and 2:
    // 4 moduli 36.6 and 37.7, 12 moduli 105.1 and 105.6; 3,211,264: 252 and 238, 756
    // and 732, 6 moduli 475 and 405).  With 2 or 3 moduli S = 1 once it is the
    // better (2 moduli, S = 2 and 1, at 200,704: 15.3 and 17.0, 400,000: 26.3 and
    // 24.8, 3,211,264: 157 and 127; 3 moduli, S = 3 and 1, at 400,000: 25.4 and
    // 29.3, 3,211,264: 173 and 165).
    uint32_t G = P.k == 2 ? 2u : 1u, S = P.k;
    if (P.n > (1u << (P.k == 3 ? 19 : 18))) {
        S = P.k <= 3 ? 1u : P.n > (1u << 19) ? 2u : 4u;
        G = S == 2 ? 2u : 4u;
    }
    hipLaunchKernelGGL(k_decode, dim3(grid_for(P.n, static_cast<int>(64 * G))), dim3(64 * G * S), 0, stream, P, C,
                       d_out_labels, d_out_zero, d_offsets, d_y, bad, G, S);
    return launched();
}

int redash_hash_labels(uint32_t q, uint32_t m, uint64_t count, const uint32_t *d_labels, uint32_t gadget_id,
                       const uint64_t *d_tau, uint32_t *d_out, hipStream_t stream) {
    if (!modulus_ok(q) || !modulus_ok(m)) return REDASH_E_PARAM;
    if (count == 0) return REDASH_OK;
    if (!d_labels || !d_tau || !d_out) return REDASH_E_NULL;
    ModConst mq, mm;
    fill_mod_const(q, &mq);
    fill_mod_const(m, &mm);
    hipLaunchKernelGGL(k_hash<256>, dim3(grid_for(count, 256)), dim3(256), 0, stream, mq, mm, count, d_labels,
                       gadget_id, d_tau, d_out);
    return launched();
}

const char *redash_strerror(int code) {
    switch (code) {
        case REDASH_OK: return "ok";
        case REDASH_E_PARAM: return "invalid parameters";
        case REDASH_E_NULL: return "null pointer";
        case REDASH_E_HIP: return "HIP launch or runtime error";
        case REDASH_E_LABEL: return "output label failed the decode check";
        case REDASH_E_SIZE: return "the call needs more working storage than the fixed buffer holds";
        default: return "unknown error";
    }
}

}  // extern "C"
