// Per-pair GateKeeper-GPU filter body for gfx950, shared by the plain and the
// mixed-batch kernels.
//
// One lane filters one (read, candidate) pair, as the paper gives one thread
// to one filtration (Sec. 3.2).  Unlike the paper's kernel, which keeps 2e+1
// masks of 2-bit-interleaved words in thread-local stack arrays, the lane:
//   - holds the read and the window as two bit-planes (high and low code bit)
//     of 32 bases per 32-bit register, so "XOR the codes, OR the two bits"
//     (Sec. 2.1) is (rh ^ gh) | (rl ^ gl) over 32 bases;
//   - gathers the window from the resident bit-plane reference with funnel
//     shifts (v_alignbit) at any base offset;
//   - never stores a mask: each of the 2e+1 masks is built and folded into one
//     running accumulator of W registers;
//   - amends without a look-up table: a 0 that stays lies in a run of three or
//     more 0s (or a run that touches an end), so each mask only contributes
//     where three 0s in a row are centred, and widening those centres back
//     into runs is done once, on what all masks of a direction collected; the
//     1s are counted with v_bcnt instead of a table.
//
// Steps per pair, all from Sec. 2.1 unless noted:
//   H        = mismatch(read, window)
//   D_k, I_k = mismatch(read shifted by +k / -k bases, window), k = 1..e;
//              vacated read positions hold code 00 (a logical shift)
//   each mask is amended: a 0-run of length 1 or 2 with a 1 on both sides
//              inside [0, m) becomes 1s (runs touching either end stay)
//   refinement (Sec. 3.4): after amendment D_k[0, k) and I_k[m-k, m) := 1
//   F        = H & AND_k (D_k & I_k);  est = popcount(F);  accept iff est <= e
// Masks with k >= m are all 1s after refinement, so k stops at min(e, m-1).
// Pairs whose read or window holds an unknown base, or whose window runs past
// the reference end, are passed as GK_UNDEFINED (Sec. 3.3).
#pragma once

#include "gk_args.h"

namespace gkd {

__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t s)
{
    // ({hi, lo} >> s)[31:0] for s in [0, 31]
    return __builtin_amdgcn_alignbit(hi, lo, s);
}

__device__ __forceinline__ uint32_t ones_below(int n)
{
    // bits [0, n) set, n clamped to [0, 32]
    n = n < 0 ? 0 : (n > 32 ? 32 : n);
    return n >= 32 ? 0xFFFFFFFFu : ((1u << n) - 1u);
}

// Three delta swaps on 16 interleaved 2-bit codes (base j in bits 2j, 2j+1):
// afterwards byte 0 holds the low code bits of bases 0-7, byte 1 their high
// bits, byte 2 the low bits of bases 8-15 and byte 3 their high bits.
__device__ __forceinline__ uint32_t unzip3(uint32_t x)
{
    uint32_t t;
    t = (x ^ (x >> 1)) & 0x22222222u; x = x ^ t ^ (t << 1);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu; x = x ^ t ^ (t << 2);
    t = (x ^ (x >> 4)) & 0x00F000F0u; x = x ^ t ^ (t << 4);
    return x;
}

// Two read words (bases 0-15 and 16-31 of a 32-base group) -> bit-planes.
template <int L>
__device__ __forceinline__ void planes_from_words(uint32_t p0, uint32_t p1, uint32_t &hi,
                                                  uint32_t &lo)
{
    if (L == GK_READS_SPLIT) {
        // low code bits in bits 0-15, high code bits in bits 16-31
        lo = __builtin_amdgcn_perm(p1, p0, 0x05040100u);
        hi = __builtin_amdgcn_perm(p1, p0, 0x07060302u);
    } else {
        const uint32_t x0 = unzip3(p0), x1 = unzip3(p1);
        lo = __builtin_amdgcn_perm(x1, x0, 0x06040200u);
        hi = __builtin_amdgcn_perm(x1, x0, 0x07050301u);
    }
}

// Amend mask M (W words, bits at or beyond m are 0) and AND (A | X) into acc.
// A 0 at position i is amended iff it lies in a 0-run of length 1 or 2 with
// 1s on both sides: M[i-1]&M[i+1] | M[i-1]&M[i+2] | M[i-2]&M[i+1].
// Positions outside [0, m) read as 0, so runs touching an end never qualify.
// Used for shifts of 32 bases and more only.
template <int W>
__device__ __forceinline__ void amend_and(const uint32_t (&M)[W], uint32_t (&acc)[W],
                                          const uint32_t (&X)[W])
{
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t prev = w > 0 ? M[w - 1] : 0u;
        const uint32_t next = w < W - 1 ? M[w + 1] : 0u;
        const uint32_t l1 = funnel(M[w], prev, 31);   // M[i-1]
        const uint32_t l2 = funnel(M[w], prev, 30);   // M[i-2]
        const uint32_t r1 = funnel(next, M[w], 1);    // M[i+1]
        const uint32_t r2 = funnel(next, M[w], 2);    // M[i+2]
        const uint32_t amended = M[w] | (l1 & (r1 | r2)) | (l2 & r1);
        acc[w] &= amended | X[w];
    }
}

template <int W>
__device__ __forceinline__ void mismatch(const uint32_t (&sh)[W], const uint32_t (&sl)[W],
                                         const uint32_t (&gh)[W], const uint32_t (&gl)[W],
                                         uint32_t (&M)[W])
{
#pragma unroll
    for (int w = 0; w < W; ++w)
        M[w] = (sh[w] ^ gh[w]) | (sl[w] ^ gl[w]);
}

// M[i-1] | M[i] | M[i+1] of word w (0 outside the words): 0 where three 0s in
// a row are centred.
template <int W>
__device__ __forceinline__ uint32_t centres(const uint32_t (&M)[W], int w)
{
    const uint32_t l1 = funnel(M[w], w > 0 ? M[w - 1] : 0u, 31);
    const uint32_t r1 = funnel(w < W - 1 ? M[w + 1] : 0u, M[w], 1);
    return M[w] | l1 | r1;
}

// x shifted up by q bits (towards higher positions); q < 32 unless ANY.
template <int W, bool ANY>
__device__ __forceinline__ void shift_up(uint32_t (&x)[W], uint32_t q)
{
    if constexpr (ANY) {
#pragma unroll
        for (int step = 8; step >= 1; step >>= 1)
            if (step < W) {
#pragma unroll
                for (int w = W - 1; w >= 0; --w)
                    x[w] = ((q >> 5) & (uint32_t)step) ? (w >= step ? x[w - step] : 0u) : x[w];
            }
    }
    const uint32_t s = q & 31u;
    if (s != 0u) {
#pragma unroll
        for (int w = W - 1; w >= 0; --w)
            x[w] = w > 0 ? funnel(x[w], x[w - 1], 32u - s) : x[0] << s;
    }
}

// x shifted down by q bits.
template <int W, bool ANY>
__device__ __forceinline__ void shift_down(uint32_t (&x)[W], uint32_t q)
{
    if constexpr (ANY) {
#pragma unroll
        for (int step = 8; step >= 1; step >>= 1)
            if (step < W) {
#pragma unroll
                for (int w = 0; w < W; ++w)
                    x[w] = ((q >> 5) & (uint32_t)step) ? (w + step < W ? x[w + step] : 0u) : x[w];
            }
    }
    const uint32_t s = q & 31u;
#pragma unroll
    for (int w = 0; w < W; ++w)
        x[w] = funnel(w < W - 1 ? x[w + 1] : 0u, x[w], s);
}

// Widens collected centres: bit i of the result is 0 iff A is 0 at i-1, i or
// i+1.  below / above: A at position -1 (bit 0 of below) and at position 32W
// (bit 31 of above).
template <int W>
__device__ __forceinline__ void widen(const uint32_t (&A)[W], uint32_t below, uint32_t above,
                                      uint32_t (&F)[W])
{
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t l1 = w > 0 ? funnel(A[w], A[w - 1], 31) : (A[0] << 1) | (below & 1u);
        const uint32_t r1 = w < W - 1 ? funnel(A[w + 1], A[w], 1)
                                      : (A[W - 1] >> 1) | (above & 0x80000000u);
        F[w] = A[w] & l1 & r1;
    }
}

// The masks of shifts 0..kmax, kmax <= min(31, m - 1), ANDed into F.  Read and
// window planes have no bits at or beyond m.  Without ANY every word but the
// top one is fully inside the read (32(W-1) < m <= 32W); with it m is any
// length up to 32W.  REFINE: the vacated positions of a shifted mask are 1
// after amendment (Sec. 3.4).
//
// VALU issue bounds the filter from about e = 6 at 100 bases up.  A mask costs
// 8 instructions per word: 2 to shift the read's planes, 2 to compare, 2 for
// the neighbours, 2 to collect (or, and bitop3).  Amending each mask by itself
// took 11 (two more neighbour funnels and one more three-input logic): the
// plain launch at 250 bases, e = 25, 2^23 pairs went from 1,023 to 734 us, at
// 150 bases, e = 7, 3 M pairs from 96 to 86 us, and at 100 bases, e = 5, where
// the window gathers bound it, stayed at 363 us (2^24 pairs).
//
// What is collected: a 0 of a mask stays 0 iff it lies in a run of at least
// three 0s, where positions outside the read count as 0s (runs touching an end
// stay), i.e. iff a centre of three 0s lies next to it or on it.  Widening
// centres into runs distributes over AND, so all masks share one pass at the
// end.  Refinement: in a deletion mask D_k only positions i >= k may stay 0.
// Centres at k+1 or higher widen into those only and are collected in A;
// centre k (0s at k-1, k, k+1) gives positions k and k+1, collected in PA, and
// centre k-1 position k, collected in PB; lower ones give nothing.  An
// insertion mask I_k is the mirror image at the read's end: for those the
// planes are shifted up so that the last base is bit 31 of the top word, which
// keeps the masks of both directions in one word and, with one k per step, in
// scalar registers.
//
// SPLIT: this lane takes shifts k0, k0 + step, ... only (F is then the AND of
// those masks and the Hamming mask).
template <int W, bool ANY, bool REFINE, bool SPLIT>
__device__ __forceinline__ void near_masks(uint32_t (&rh)[W], uint32_t (&rl)[W],
                                           uint32_t (&gh)[W], uint32_t (&gl)[W], uint32_t m,
                                           uint32_t kmax, uint32_t (&F)[W], uint32_t k0,
                                           uint32_t step)
{
    const uint32_t kfirst = SPLIT ? k0 : 1u, kstep = SPLIT ? step : 1u;
    uint32_t A[W], M[W], sh[W], sl[W];
    mismatch<W>(rh, rl, gh, gl, M);            // Hamming mask (never refined)
    uint32_t first = M[0], last = M[W - 1];    // mask bits 0 and 32W - 1 (centres -1 and 32W)
#pragma unroll
    for (int w = 0; w < W; ++w)
        A[w] = centres<W>(M, w);

    // Deletion masks: read[i-k] against window[i].
    uint32_t PA = 0xFFFFFFFFu, PB = 0xFFFFFFFFu;
    const uint32_t vtop = ones_below((int)m - 32 * (W - 1));
    for (uint32_t k = kfirst; k <= kmax; k += kstep) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sh[w] = w > 0 ? funnel(rh[w], rh[w - 1], 32u - k) : (rh[0] << k);
            sl[w] = w > 0 ? funnel(rl[w], rl[w - 1], 32u - k) : (rl[0] << k);
        }
        mismatch<W>(sh, sl, gh, gl, M);
        if constexpr (ANY) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                M[w] &= ones_below((int)m - 32 * w);
        } else {
            M[W - 1] &= vtop;                  // bases moved past the read end
        }
        last &= M[W - 1];
        if constexpr (!REFINE)
            first &= M[0];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t c = centres<W>(M, w);
            if (REFINE && w == 0) {
                A[0] &= c | ((2u << k) - 1u);
                PA &= c | ~(1u << k);
                PB &= c | ~(1u << (k - 1u));
            } else {
                A[w] &= c;
            }
        }
    }
    widen<W>(A, first, last, F);
    if constexpr (REFINE) {
        F[0] &= PA & ((PA << 1) | 1u) & ((PB << 1) | 1u);
        if constexpr (W >= 2)
            F[1] &= (PA >> 31) | ~1u;
    }

    // Insertion masks: read[i+k] against window[i], last base in bit 31 of
    // word W-1, first base in bit q.
    const uint32_t q = 32u * W - m;
    shift_up<W, ANY>(rh, q);
    shift_up<W, ANY>(rl, q);
    shift_up<W, ANY>(gh, q);
    shift_up<W, ANY>(gl, q);
    PA = PB = first = last = 0xFFFFFFFFu;
#pragma unroll
    for (int w = 0; w < W; ++w)
        A[w] = 0xFFFFFFFFu;
    const uint32_t vlow = 0xFFFFFFFFu << (q & 31u);
    for (uint32_t k = kfirst; k <= kmax; k += kstep) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sh[w] = w < W - 1 ? funnel(rh[w + 1], rh[w], k) : (rh[W - 1] >> k);
            sl[w] = w < W - 1 ? funnel(rl[w + 1], rl[w], k) : (rl[W - 1] >> k);
        }
        mismatch<W>(sh, sl, gh, gl, M);
        if constexpr (ANY) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                M[w] &= ~ones_below((int)q - 32 * w);
        } else {
            M[0] &= vlow;                      // bases moved past the read start
        }
        first &= M[0];
        if constexpr (!REFINE)
            last &= M[W - 1];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t c = centres<W>(M, w);
            if (REFINE && w == W - 1) {
                A[W - 1] &= c | (0xFFFFFFFFu << (31u - k));
                PA &= c | ~(1u << (31u - k));
                PB &= c | ~(1u << (32u - k));
            } else {
                A[w] &= c;
            }
        }
    }
    uint32_t G[W];
    widen<W>(A, first, last, G);
    if constexpr (REFINE) {
        G[W - 1] &= PA & ((PA >> 1) | 0x80000000u) & ((PB >> 1) | 0x80000000u);
        if constexpr (W >= 2)
            G[W - 2] &= (PA << 31) | 0x7FFFFFFFu;
    }
    shift_down<W, ANY>(G, q);
#pragma unroll
    for (int w = 0; w < W; ++w)
        F[w] &= G[w];
}

// ---- masks of up to BLOCK_KMAX shifts in blocks of 64 bits ------------------
//
// near_masks spends two of its eight instructions per word on the neighbours
// M[i-1] and M[i+1], a funnel shift each.  A 64-bit shift by a constant issues
// at the rate of a 32-bit one (35 T lanes/s both), so on blocks of two words
// the neighbours cost half, if no bit has to come from another block.  Blocks
// therefore overlap by two bits: word w starts at position 32w - w_off(w), and
// centres are collected at the position of their last (deletions) or first
// (insertions) base, so that the bits a block lacks are the ones its neighbour
// has.  The words then hold block_cap positions: 64, 126, 188, 250 ... of an
// even number of words.  2^23 pairs of 250 bases at e = 25 went from 737 to 699 us, a
// mixed batch of 2^24 pairs (64 to 300 bases) from 785 to 776.  Reads of the last
// few lengths of a word count (127, 128, 157-160, 251-256, ...) stay with near_masks.
//
// Laying out the blocks and going back costs about 11 instructions per word,
// and a shift (two masks) saves two per word, less two: from 7 shifts on at 8
// words, 9 at 5.  With every wave on blocks 250 bases at e = 25 gained 4.7% and
// 150 at e = 7 or 100 at e = 5 lost 1.3%, so a wave takes them from BLOCK_KMIN
// shifts on, if all its pairs fit (lanes on both ways would run both).  Lanes
// that share a pair's shifts have too few each.
constexpr uint32_t BLOCK_KMAX = 30;          // shifts whose edges fit one word
constexpr uint32_t BLOCK_KMIN = 10;
constexpr int BLOCK_WMIN = 4;

__host__ __device__ constexpr uint32_t w_off(int w) { return 2u * (uint32_t)(w / 2); }

template <int W>
__device__ __forceinline__ constexpr uint32_t block_cap()
{
    return 32u * W - w_off(W - 1);
}

// Plane words to block words.
template <int W>
__device__ __forceinline__ void to_blocks(uint32_t (&x)[W])
{
#pragma unroll
    for (int w = W - 1; w >= 2; --w)
        x[w] = funnel(x[w], x[w - 1], 32u - w_off(w));
}

// The 32 positions below block word w >= 1, and the 32 above it.
template <int W>
__device__ __forceinline__ uint32_t below(const uint32_t (&x)[W], int w)
{
    return w % 2 ? x[w - 1] : funnel(x[w - 1], x[w - 2], 30);
}

template <int W>
__device__ __forceinline__ uint32_t above(const uint32_t (&x)[W], int w)
{
    if (w == W - 1)
        return 0u;
    return w % 2 ? funnel(w + 2 < W ? x[w + 2] : 0u, x[w + 1], 2) : x[w + 1];
}

// Block words shifted up by q < 32 positions.
template <int W>
__device__ __forceinline__ void blocks_up(uint32_t (&x)[W], uint32_t q)
{
    if (q != 0u) {
#pragma unroll
        for (int w = W - 1; w >= 1; --w)
            x[w] = funnel(x[w], below<W>(x, w), 32u - q);
        x[0] <<= q;
    }
}

// M of the next position below (UP) or above in the block, and of the one after.
template <int W, bool UP>
__device__ __forceinline__ void block_centres(const uint32_t (&M)[W], uint32_t (&one)[W],
                                              uint32_t (&two)[W])
{
    // (opaque: a right shift by a constant becomes a funnel and a shift)
    uint32_t by1 = 1u, by2 = 2u;
    asm("" : "+s"(by1), "+s"(by2));
#pragma unroll
    for (int w = 0; w + 1 < W; w += 2) {
        const uint64_t x = (uint64_t)M[w + 1] << 32 | M[w];
        const uint64_t y = UP ? x << 1 : x >> by1, z = UP ? x << 2 : x >> by2;
        one[w] = (uint32_t)y;
        one[w + 1] = (uint32_t)(y >> 32);
        two[w] = (uint32_t)z;
        two[w + 1] = (uint32_t)(z >> 32);
    }
    if constexpr (W % 2) {
        one[W - 1] = UP ? M[W - 1] << 1 : M[W - 1] >> 1;
        two[W - 1] = UP ? M[W - 1] << 2 : M[W - 1] >> 2;
    }
}

// near_masks with refinement, for 32(W-1) < m <= block_cap and
// kmax <= min(BLOCK_KMAX, m - 1).
template <int W>
__device__ __forceinline__ void block_masks(uint32_t (&rh)[W], uint32_t (&rl)[W],
                                            uint32_t (&gh)[W], uint32_t (&gl)[W], uint32_t m,
                                            uint32_t kmax, uint32_t (&F)[W])
{
    constexpr uint32_t OFF = w_off(W - 1);
    uint32_t A[W], M[W], one[W], two[W], sh[W], sl[W], nh[W], nl[W];
    to_blocks<W>(rh);
    to_blocks<W>(rl);
    to_blocks<W>(gh);
    to_blocks<W>(gl);

    // Hamming and deletion masks: read[i-k] against window[i], centre i at bit
    // i + 1.  Above the top word: centres block_cap - 1 (tail) and block_cap (last).
    mismatch<W>(rh, rl, gh, gl, M);
    block_centres<W, true>(M, one, two);
    uint32_t last = M[W - 1], tail = M[W - 1] | one[W - 1];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        A[w] = M[w] | one[w] | two[w];
        nh[w] = w > 0 ? below<W>(rh, w) : 0u;
        nl[w] = w > 0 ? below<W>(rl, w) : 0u;
    }
    uint32_t PA = 0xFFFFFFFFu, PB = 0xFFFFFFFFu;
    const uint32_t vtop = ones_below((int)m - 32 * (W - 1) + (int)OFF);
    for (uint32_t k = 1; k <= kmax; ++k) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sh[w] = w > 0 ? funnel(rh[w], nh[w], 32u - k) : rh[0] << k;
            sl[w] = w > 0 ? funnel(rl[w], nl[w], 32u - k) : rl[0] << k;
        }
        mismatch<W>(sh, sl, gh, gl, M);
        M[W - 1] &= vtop;                      // bases moved past the read end
        last &= M[W - 1];
        block_centres<W, true>(M, one, two);
        tail &= M[W - 1] | one[W - 1];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t c = M[w] | one[w] | two[w];
            if (w == 0) {
                A[0] &= c | ((4u << k) - 1u);
                PA &= c | ~(2u << k);
                PB &= c | ~(1u << k);
            } else {
                A[w] &= c;
            }
        }
    }
    {   // back to plane words, then widened: F[i] = A[i] & A[i+1] & A[i+2]
        const uint32_t over = tail >> 31 | (last >> 31) << 1;
        uint32_t a[W + 1];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t next = w == W - 1 ? over : w % 2 ? A[w + 1] >> 2 : A[w + 1];
            a[w] = funnel(next, A[w], w_off(w));
        }
        a[W] = OFF == 0u ? over : 0u;
#pragma unroll
        for (int w = 0; w < W; ++w)
            F[w] = a[w] & funnel(a[w + 1], a[w], 1) & funnel(a[w + 1], a[w], 2);
        F[0] &= PA & (PA >> 1 | 0x80000000u) & PB;
    }

    // Insertion masks: read[i+k] against window[i], last base at block_cap - 1,
    // first base in bit q, centre i at bit i - 1.  Below bit 0: centres 0
    // (head) and -1 (first).
    const uint32_t q = block_cap<W>() - m;
    blocks_up<W>(rh, q);
    blocks_up<W>(rl, q);
    blocks_up<W>(gh, q);
    blocks_up<W>(gl, q);
    uint32_t head = 0xFFFFFFFFu, first = 0xFFFFFFFFu;
    PA = PB = 0xFFFFFFFFu;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        A[w] = 0xFFFFFFFFu;
        nh[w] = above<W>(rh, w);
        nl[w] = above<W>(rl, w);
    }
    const uint32_t vlow = 0xFFFFFFFFu << q;
    for (uint32_t k = 1; k <= kmax; ++k) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sh[w] = w < W - 1 ? funnel(nh[w], rh[w], k) : rh[W - 1] >> k;
            sl[w] = w < W - 1 ? funnel(nl[w], rl[w], k) : rl[W - 1] >> k;
        }
        mismatch<W>(sh, sl, gh, gl, M);
        M[0] &= vlow;                          // bases moved past the read start
        first &= M[0];
        block_centres<W, false>(M, one, two);
        head &= M[0] | one[0];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t c = M[w] | one[w] | two[w];
            if (w == W - 1) {
                A[W - 1] &= c | (0xFFFFFFFFu << (30u - k));
                PA &= c | ~(1u << (30u - k));
                PB &= c | ~(1u << (31u - k));
            } else {
                A[w] &= c;
            }
        }
    }
    uint32_t G[W];
    {   // G[i] = A[i] & A[i-1] & A[i-2]
        uint32_t a[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (w % 2 && w < W - 1)
                a[w] = funnel(A[w + 1] >> 2, (A[w] & 0x3FFFFFFFu) | A[w + 1] << 30, w_off(w));
            else
                a[w] = funnel(w < W - 1 ? A[w + 1] : 0u, A[w], w_off(w));
        }
        const uint32_t under = head << 31 | (first & 1u) << 30;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t prev = w > 0 ? a[w - 1] : under;
            G[w] = a[w] & funnel(a[w], prev, 31) & funnel(a[w], prev, 30);
        }
        const uint32_t R = PA & (PA << 1 | 1u) & PB;
        G[W - 1] &= OFF == 0u ? R : funnel(0xFFFFFFFFu, R, OFF);
        if constexpr (OFF != 0u)
            G[W - 2] &= funnel(R, 0xFFFFFFFFu, OFF);
    }
    shift_down<W, false>(G, q);
#pragma unroll
    for (int w = 0; w < W; ++w)
        F[w] &= G[w];
}

// Read r's plane words 0..W-1 from global memory (words at or beyond the read
// length are 0), for the general path.
template <int W, int L>
__device__ __forceinline__ void load_read(const FilterArgs &a, uint32_t r, uint32_t m,
                                          uint32_t (&rh)[W], uint32_t (&rl)[W])
{
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t *row0 = a.reads + (size_t)(2 * w) * a.pitch;
        const uint32_t *row1 = a.reads + (size_t)(2 * w + 1) * a.pitch;
        const uint32_t p0 = (m > 32u * w) ? row0[r] : 0u;
        const uint32_t p1 = (m > 32u * w + 16u) ? row1[r] : 0u;
        planes_from_words<L>(p0, p1, rh[w], rl[w]);
    }
}

// General path: any m <= 32W and any k <= m-1 <= 511, in acc (bits at or
// beyond m are 0).  Shifts below 32 as near_masks; from 32 bases on whole
// words move: the read planes are shifted in place by one word each time k
// passes a multiple of 32, each mask is amended by itself, and the planes are
// rebuilt between the deletion and the insertion loop: reloaded from the read
// rows in memory, or, with KEPT (reads that exist only in registers), taken
// again from the pair's words.
template <int W, int L, bool REFINE, bool KEPT, bool SPLIT>
__device__ __forceinline__ void general_masks(const FilterArgs &a, uint32_t r,
                                              const uint32_t (&words)[2 * W], uint32_t (&rh)[W],
                                              uint32_t (&rl)[W], uint32_t (&gh)[W],
                                              uint32_t (&gl)[W], uint32_t m, uint32_t kmax,
                                              uint32_t (&acc)[W], uint32_t k0, uint32_t step)
{
    uint32_t V[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        V[w] = ones_below((int)m - 32 * w);
        rh[w] &= V[w];
        rl[w] &= V[w];
        gh[w] &= V[w];
        gl[w] &= V[w];
    }
    near_masks<W, true, REFINE, SPLIT>(rh, rl, gh, gl, m, kmax < 31u ? kmax : 31u, acc, k0, step);

    if (W > 1 && kmax > 31u) {
        const uint32_t q = 32u * W - m;
        shift_down<W, true>(rh, q);
        shift_down<W, true>(rl, q);
        shift_down<W, true>(gh, q);
        shift_down<W, true>(gl, q);
        uint32_t M[W], X[W], sh[W], sl[W];
        for (uint32_t k = 32; k <= kmax; ++k) {
            if (((k - 1) & 31u) == 0u) {           // read moves up one more word
#pragma unroll
                for (int w = W - 1; w >= 0; --w) {
                    rh[w] = w > 0 ? rh[w - 1] : 0u;
                    rl[w] = w > 0 ? rl[w - 1] : 0u;
                }
            }
            const uint32_t s = 32u - (k - ((k - 1) & ~31u));  // in [0, 31]
#pragma unroll
            for (int w = 0; w < W; ++w) {
                sh[w] = funnel(rh[w], w > 0 ? rh[w - 1] : 0u, s);
                sl[w] = funnel(rl[w], w > 0 ? rl[w - 1] : 0u, s);
            }
            mismatch<W>(sh, sl, gh, gl, M);
#pragma unroll
            for (int w = 0; w < W; ++w) {
                M[w] &= V[w];
                X[w] = REFINE ? ones_below((int)k - 32 * w) : 0u;
            }
            amend_and<W>(M, acc, X);
        }

        if constexpr (KEPT) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                planes_from_words<L>(words[2 * w], words[2 * w + 1], rh[w], rl[w]);
        } else {
            load_read<W, L>(a, r, m, rh, rl);
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            rh[w] &= V[w];
            rl[w] &= V[w];
        }
        for (uint32_t k = 32; k <= kmax; ++k) {
            if ((k & 31u) == 0u) {                 // read moves down one more word
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    rh[w] = w < W - 1 ? rh[w + 1] : 0u;
                    rl[w] = w < W - 1 ? rl[w + 1] : 0u;
                }
            }
            const uint32_t s = k & 31u;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                sh[w] = funnel(w < W - 1 ? rh[w + 1] : 0u, rh[w], s);
                sl[w] = funnel(w < W - 1 ? rl[w + 1] : 0u, rl[w], s);
            }
            mismatch<W>(sh, sl, gh, gl, M);
#pragma unroll
            for (int w = 0; w < W; ++w)
                X[w] = REFINE ? V[w] & ~ones_below((int)m - (int)k - 32 * w) : 0u;
            amend_and<W>(M, acc, X);
        }
    }
#pragma unroll
    for (int w = 0; w < W; ++w)
        acc[w] &= V[w];
}

// Indices of one pair (first-level loads).
struct PairIdx {
    uint32_t r, pos, e;
};

// Second-level loads of one pair: read length and unknown flag, read words,
// window words, and the words of the unknown-line summary that cover the
// window.  Issued speculatively (indices clamped into range) so that they can
// be in flight before the pair's validity is known, and without a branch
// around any one load: at a branch the compiler waits for what is in flight.
template <int W>
struct PairData {
    uint32_t m, has_n;
    uint32_t unk0, unk1;        // summary words of the window's first and last line
    uint32_t words[2 * W];
    uint4 win[(W + 3) / 2];     // pairs of plane words from an even word on
};

// Plain loads throughout: marking the read words and pair entries that are used
// once as non-temporal moved the 100-base launch by 0.7% and no other.

// base[i] for i < 2^30 (reads, and the pairs of a launch) of elements of up to
// 4 bytes: a 32-bit offset from a scalar base, no 64-bit address per lane.
// With the window loads by one base for both copies of the planes, that is 2%
// fewer vector instructions per pair: 2^23 pairs of 250 bases at e = 25 went from
// 746 to 736 us, a mixed batch of 2^24 (64 to 300 bases) from 807 to 789.
template <typename T>
__device__ __forceinline__ T elem(const T *base, uint32_t i)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) +
                                        (uint32_t)(i * (uint32_t)sizeof(T)));
}

template <typename T>
__device__ __forceinline__ void put(T *base, uint32_t i, T v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<T *>(reinterpret_cast<char *>(base) +
                                                         (uint32_t)(i * (uint32_t)sizeof(T))));
}

__device__ __forceinline__ PairIdx load_idx(const FilterArgs &a, uint32_t i)
{
    PairIdx p;
    p.r = a.pair_read ? elem(a.pair_read, i) : i;
    p.pos = elem(a.cand_pos, i);
    p.e = a.e_pair ? (uint32_t)elem(a.e_pair, i) : a.e_uniform;
    return p;
}

// The window words of a pair: only those a window of up to max_read_len
// bases can touch, from the copy of the planes in which they share one
// 128-byte line, as aligned pairs of words.
//
// The line rate bounds these gathers (a random line per pair), and every
// further load of a line is another look-up, by which time the line may have
// left the L1: three aligned 16-byte loads per window of 100 bases ran 66.6 G
// windows/s over a 25 MB reference and 52.4 G over 775 MB, five 8-byte loads
// 60.2 G and 38.3 G.  With every load of a pair in flight at once (reads first:
// they need no position) the plain launch went from 363 to 345 us for 2^24
// pairs of 100 bases, 84 lines per 64 pairs at 64 G lines/s.
template <int W>
__device__ __forceinline__ uint32_t longest(const FilterArgs &a)
{
    return a.max_read_len < 32u * W ? a.max_read_len : 32u * W;
}

template <int W>
__device__ __forceinline__ void load_window(const FilterArgs &a, uint32_t pos, PairData<W> &d)
{
    pos = pos < a.ref_len ? pos : 0u;
    const uint32_t w0 = pos >> 5;
    const uint32_t nw = ((pos & 31u) + longest<W>(a) + 31u) >> 5;
    const bool use_b = (w0 >= REF_SHIFT_WORDS) & ((w0 & (LINE_WORDS - 1u)) + nw > LINE_WORDS);
    // REF_SHIFT_WORDS is even: an even word of one copy is one of the other
    // (words of both copies number less than 2^29: a 32-bit byte offset)
    const char *planes = reinterpret_cast<const char *>(a.ref_planes);
    const uint32_t first = ((use_b ? w0 + a.ref_b_words - REF_SHIFT_WORDS : w0) & ~1u) * 8u;
    // A pair of words the window does not reach is replaced by its last one (no
    // branch, no other line); its bases lie beyond every read's end.
    const uint32_t last = ((pos & 63u) + longest<W>(a) - 1u) >> 6;
#pragma unroll
    for (int j = 0; j < (W + 3) / 2; ++j)
        d.win[j] = *reinterpret_cast<const uint4 *>(
            planes + (uint32_t)(first + 16u * ((uint32_t)j < last ? (uint32_t)j : last)));
}

template <int W>
__device__ __forceinline__ void load_unknown_lines(const FilterArgs &a, uint32_t pos,
                                                   PairData<W> &d)
{
    d.unk0 = d.unk1 = 0u;
    if (a.ref_has_unknown) {
        pos = pos < a.ref_len ? pos : 0u;
        const uint32_t *lines = reinterpret_cast<const uint32_t *>(a.ref_unk_lines);
        d.unk0 = elem(lines, pos / LINE_BASES >> 5);
        d.unk1 = elem(lines, (uint32_t)(((uint64_t)pos + longest<W>(a) - 1u) / LINE_BASES >> 5));
    }
}

// A row beyond the last repeats it: its bases lie beyond every read's end.
// With no reads the host points reads and read_len at memory that may be
// read (pitch 0), and pair_gate ignores what comes.
template <int W>
__device__ __forceinline__ void load_words(const FilterArgs &a, uint32_t r, PairData<W> &d)
{
#pragma unroll
    for (int j = 0; j < 2 * W; ++j) {
        const uint32_t row = (uint32_t)j < a.rows ? (uint32_t)j : a.rows - 1u;
        d.words[j] = elem(a.reads + (size_t)row * a.pitch, r);
    }
}

// The same from reads in rows of a.pitch words (a multiple of 4), one run of
// 16-byte loads per read.
template <int W>
__device__ __forceinline__ void load_words_rowwise(const FilterArgs &a, uint32_t r, PairData<W> &d)
{
    const uint4 *q = reinterpret_cast<const uint4 *>(a.reads + (size_t)r * a.pitch);
#pragma unroll
    for (int j = 0; j < 2 * W; j += 4) {
        const uint4 v = q[(uint32_t)j < a.pitch ? (uint32_t)j / 4u : a.pitch / 4u - 1u];
        const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j + k < 2 * W)
                d.words[j + k] = w4[k];
    }
}

template <int W, bool ROWWISE = false>
__device__ __forceinline__ void load_data(const FilterArgs &a, const PairIdx &p, PairData<W> &d)
{
    const uint32_t r = p.r < a.n_reads ? p.r : 0u;
    if constexpr (ROWWISE)
        load_words_rowwise<W>(a, r, d);
    else
        load_words<W>(a, r, d);
    const uint8_t *flag = a.read_has_n ? a.read_has_n
                                       : reinterpret_cast<const uint8_t *>(a.read_len);
    d.m = (uint32_t)elem(a.read_len, r);
    d.has_n = (uint32_t)elem(flag, r);
    load_window<W>(a, p.pos, d);
    load_unknown_lines<W>(a, p.pos, d);
}

// Whether a pair whose loads have arrived can be compared (Sec. 3.3): returns
// PAIR_OK and sets m, or GK_INVALID (read length 0 or above max_read_len, or
// no such read) or GK_UNDEFINED (an unknown base in the read or the window, or
// a window past the reference end).
constexpr uint32_t PAIR_OK = 0xFFu;

template <int W>
__device__ __forceinline__ uint32_t pair_gate(const FilterArgs &a, const PairIdx &p,
                                              const PairData<W> &d, uint32_t &m)
{
    m = p.r < a.n_reads ? d.m : 0u;
    if (m == 0u || m > a.max_read_len)
        return GK_INVALID;
    if ((uint64_t)p.pos + m > a.ref_len || (a.read_has_n && d.has_n))
        return GK_UNDEFINED;
    if (a.ref_has_unknown) {
        // Only windows touching a 512-base line that holds an unknown base
        // read the unknown plane (reads have at most 512 bases, so at most two lines).
        const uint32_t l0 = p.pos / LINE_BASES;
        const uint32_t l1 = (uint32_t)(((uint64_t)p.pos + longest<W>(a) - 1u) / LINE_BASES);
        if ((((d.unk0 >> (l0 & 31u)) | (d.unk1 >> (l1 & 31u))) & 1u) == 0u)
            return PAIR_OK;
        const uint32_t s = p.pos & 31u;
        const uint32_t *u = a.ref_unk + (p.pos >> 5);
        uint32_t any = 0, cu = u[0];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t nu = u[w + 1];
            any |= funnel(nu, cu, s) & ones_below((int)m - 32 * w);
            cu = nu;
        }
        if (any)
            return GK_UNDEFINED;
    }
    return PAIR_OK;
}

// Read and window bit-planes of a pair that passed pair_gate, the window words
// funnel-shifted by pos mod 32.  Bits at or beyond m are left as they come.
template <int W, int L>
__device__ __forceinline__ void pair_planes(const PairIdx &p, const PairData<W> &d,
                                            uint32_t (&gh)[W], uint32_t (&gl)[W],
                                            uint32_t (&rh)[W], uint32_t (&rl)[W])
{
    const uint32_t s = p.pos & 31u;
    const bool odd = (p.pos & 32u) != 0u;
    uint2 win[W + 1];
#pragma unroll
    for (int w = 0; w <= W; ++w) {
        const uint4 here = d.win[w / 2], next = d.win[w / 2 + 1 < (W + 3) / 2 ? w / 2 + 1 : w / 2];
        const uint2 even_w = w % 2 ? make_uint2(here.z, here.w) : make_uint2(here.x, here.y);
        const uint2 odd_w = w % 2 ? make_uint2(next.x, next.y) : make_uint2(here.z, here.w);
        win[w] = odd ? odd_w : even_w;
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        gh[w] = funnel(win[w + 1].x, win[w].x, s);
        gl[w] = funnel(win[w + 1].y, win[w].y, s);
        planes_from_words<L>(d.words[2 * w], d.words[2 * w + 1], rh[w], rl[w]);
    }
}

// Filter one pair whose loads have arrived: returns the result code and sets
// est (GK_EST_NONE unless REJECT / ACCEPT).  With GENERAL false the caller
// guarantees 32(W-1) < m <= 32W and min(e, m-1) <= 31 for every valid pair,
// and only the register-light fast path is compiled.  VAR compiles the
// variant semantics of a.flags (GK_FLAG_*); without it a.flags must be 0, and
// the paper's filter is the only code in the kernel.  KEPT: the read has no
// rows in memory (a.reads is not used), and the general path rebuilds its
// planes from d.words.  SPLIT: `lanes` neighbouring lanes (2, 4 or 8, aligned)
// hold the same pair and take its shifts in turn, lane `sub` of them from
// sub + 1 on; all return the result.
template <int W, int L, bool GENERAL = true, bool VAR = false, bool KEPT = false,
          bool SPLIT = false>
__device__ __forceinline__ uint32_t compute_pair(const FilterArgs &a, const PairIdx &p,
                                                 const PairData<W> &d, uint32_t &est,
                                                 uint32_t sub = 0, uint32_t lanes = 1)
{
    est = GK_EST_NONE;
    uint32_t m;
    const uint32_t gate = pair_gate<W>(a, p, d, m);
    if (gate != PAIR_OK)
        return gate;
    uint32_t gh[W], gl[W], rh[W], rl[W], F[W];
    pair_planes<W, L>(p, d, gh, gl, rh, rl);
    const uint32_t kmax = p.e < m - 1u ? p.e : m - 1u;
    const bool exact = !GENERAL || (m > 32u * (W - 1) && kmax <= 31u);
    const uint32_t vtop = ones_below((int)m - 32 * (W - 1));
    if (exact) {
        rh[W - 1] &= vtop;
        rl[W - 1] &= vtop;
        gh[W - 1] &= vtop;
        gl[W - 1] &= vtop;
    }
    bool refine = true;
    if constexpr (VAR) {                       // variants (uniform per launch)
        if (a.flags & GK_FLAG_HAMMING_FASTPATH) {
            uint32_t hd = 0;
#pragma unroll
            for (int w = 0; w < W; ++w)
                hd += __builtin_popcount(((rh[w] ^ gh[w]) | (rl[w] ^ gl[w])) &
                                         ones_below((int)m - 32 * w));
            if (hd <= p.e) {
                est = hd;
                return GK_ACCEPT;
            }
        }
        if (a.flags & GK_FLAG_NO_REFINE) {
            refine = false;
            if (exact)
                near_masks<W, false, false, SPLIT>(rh, rl, gh, gl, m, kmax, F, sub + 1u, lanes);
            else
                general_masks<W, L, false, KEPT, SPLIT>(a, p.r, d.words, rh, rl, gh, gl, m, kmax,
                                                        F, sub + 1u, lanes);
        }
    }
    if (refine) {
        uint32_t blocks = 0u;
        if constexpr (W >= BLOCK_WMIN && !SPLIT) {   // (one way for the whole wave)
            blocks = __ballot(!(exact && m <= block_cap<W>() && kmax <= BLOCK_KMAX)) == 0ull &&
                     __ballot(kmax >= BLOCK_KMIN) != 0ull;
            // (opaque: a branch known to be uniform took 25 more registers)
            asm("" : "+v"(blocks));
        }
        if (blocks != 0u)
            block_masks<W>(rh, rl, gh, gl, m, kmax, F);
        else if (exact)
            near_masks<W, false, true, SPLIT>(rh, rl, gh, gl, m, kmax, F, sub + 1u, lanes);
        else
            general_masks<W, L, true, KEPT, SPLIT>(a, p.r, d.words, rh, rl, gh, gl, m, kmax, F,
                                                   sub + 1u, lanes);
    }
    if constexpr (SPLIT) {
        for (uint32_t o = 1; o < lanes; o <<= 1) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                F[w] &= __shfl_xor(F[w], (int)o, 64);
        }
    }
    if (exact)
        F[W - 1] &= vtop;
    est = 0;
#pragma unroll
    for (int w = 0; w < W; ++w)
        est += __builtin_popcount(F[w]);
    return est <= p.e ? GK_ACCEPT : GK_REJECT;
}

// Bits 0, step, 2 step, ... of x (step a power of two, the others 0), moved
// together.
__device__ __forceinline__ unsigned long long gather_bits(unsigned long long x, uint32_t step)
{
    // groups of `width` bits lie at multiples of width * step: join neighbours
    for (uint32_t width = 1; width * step < 64u; width <<= 1) {
        const uint32_t dist = width * step;
        const unsigned long long group = (1ull << width) - 1ull;
        unsigned long long y = 0;
        for (uint32_t at = 0; at < 64u; at += 2u * dist)
            y |= (x >> at & group) << at | (x >> (at + dist) & group) << (at + width);
        x = y;
    }
    return x;
}

// Accept bits of a wave that holds 64 >> lg pairs, 2^lg lanes (2, 4 or 8) to
// each; i: the lane's pair, on: its bit, on the first of its lanes only.  The
// grid holds every bit of the bitmap's words, and whole workgroups of it: with
// two lanes per pair a workgroup is two words wide, and the second word of the
// last one may lie past the bitmap.
__device__ __forceinline__ void store_split_bits(const FilterArgs &a, uint32_t i, uint32_t lg,
                                                 bool on)
{
    const unsigned long long bits = gather_bits(__ballot(on), 1u << lg);
    const uint32_t end = ((uint32_t)a.n_pairs + 63u) & ~63u;
    if ((threadIdx.x & 63u) == 0u && i < end) {
        if (lg == 1u)
            reinterpret_cast<uint32_t *>(a.accept_bits)[i >> 5] = (uint32_t)bits;
        else if (lg == 2u)
            reinterpret_cast<uint16_t *>(a.accept_bits)[i >> 4] = (uint16_t)bits;
        else
            reinterpret_cast<uint8_t *>(a.accept_bits)[i >> 3] = (uint8_t)bits;
    }
}

}  // namespace gkd
