// Kernel-facing declarations of libgk: the resident reference layout and the
// argument blocks the filter kernels take (host-only state is in
// gk_internal.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gk.h"

// Resident reference layout (device):
//   planes[j].x : bit b = high bit of the 2-bit code of base 32j+b
//   planes[j].y : bit b = low bit of the 2-bit code of base 32j+b
//   unknown[j]  : bit b = 1 iff base 32j+b is not A/C/G/T
// Bases at or beyond the reference length are 0 in all three.  REF_PAD_WORDS
// zero words follow the last word so that a window gather of up to
// GK_MAX_READ_LEN/32 + 1 words from any in-range window start stays inside
// the allocation.
namespace gkd {
constexpr uint32_t REF_PAD_WORDS = 32;
constexpr uint32_t MAX_WORDS = GK_MAX_READ_LEN / 32;  // 32-base words per mask
constexpr uint32_t GK_PPL_RESIDENT = 65536;  // pairs-per-lane value meaning
                                             // "one residency of the device"

// Second copy of the planes, shifted by half a 128-byte cache line:
// word j of the copy is ref_planes[j + REF_SHIFT_WORDS].  A window gather of up
// to 9 words that crosses a line of ref_planes lies within one line of the
// copy, so every window of up to 256 bases costs one line fetch.  The copy
// follows in the same allocation, ref_b_words (a multiple of 16) words on.
constexpr uint32_t LINE_WORDS = 16;          // uint2 words per 128-byte line
constexpr uint32_t LINE_BASES = 32 * LINE_WORDS;
constexpr uint32_t REF_SHIFT_WORDS = 8;

struct FilterArgs {
    const uint2 *ref_planes;
    const uint32_t *ref_unk;
    const unsigned long long *ref_unk_lines;  // bit L: bases [512 L, 512 L + 512)
                                              // hold an unknown base
    uint64_t ref_len;
    uint32_t ref_has_unknown;
    uint32_t ref_b_words;       // where the shifted copy begins
    uint32_t n_reads;
    uint32_t pitch;
    uint32_t e_uniform;
    uint32_t max_read_len;      // reads longer than this are GK_INVALID: the
                                // read rows hold ceil(max_read_len/16) words
    uint32_t rows;              // ceil(max_read_len / 16)
    uint32_t flags;             // GK_FLAG_* variant semantics (0: the paper's)
    const uint32_t *reads;
    const uint16_t *read_len;
    const uint8_t *read_has_n;
    const uint32_t *pair_read;
    const uint32_t *cand_pos;
    const uint8_t *e_pair;
    uint64_t n_pairs;
    uint8_t *accept;
    uint16_t *est;
    unsigned long long *accept_bits;
};

// A table of batches filtered by one persistent launch (the serving loop's
// tick): batch b owns the launch's tiles [prefix[b], prefix[b+1]).
constexpr uint32_t MAX_TABLE_BATCHES = 256;
struct BatchTable {
    uint32_t n_batches;
    uint32_t pad_[3];
    uint32_t prefix[MAX_TABLE_BATCHES + 1];
    FilterArgs args[MAX_TABLE_BATCHES];
};

// Lanes per pair (log2) of a small batch: below one wave per SIMD (65,536
// lanes) a launch takes as long as its slowest lane, whose time is its chain of
// masks, so the masks are shared out.  e: the threshold, or where each pair has
// its own the one that a tenth of the longest read would have.  Sharing costs
// about 1 us (masks by lane, the AND across lanes).  250 bases, e = 25: 11.3
// -> 5.4 us with 8 lanes (8,192 pairs), 11.5 -> 6.5 with 4 (16,384), 11.5 -> 9.0
// with 2 (32,768); 150 bases, e = 7: 5.0 -> 3.9, 5.1 -> 4.3 and 5.1 -> 5.3; 100
// bases, e = 5: 3.7 -> 3.6, 3.7 -> 4.0.
inline uint32_t split_lanes(uint64_t n_pairs, uint32_t e, uint32_t words)
{
    const uint32_t work = (e < 31u ? e : 31u) * words;
    if (n_pairs <= 12288)
        return work >= 30u ? 3u : 0u;
    if (n_pairs <= 24576)
        return work >= 30u ? 2u : 0u;
    return n_pairs <= 49152 && work >= 100u ? 1u : 0u;
}

// Pairs per tile of the mixed launch for a value of GK_OPT_MIXED_TILE.
inline uint32_t mixed_tile(uint32_t option) { return option / 4; }

// Pairs per tile where no tuning was set.  A small batch needs tiles enough
// for every compute unit (60,001 mixed pairs over 3.1 Gbp: 18 us with 256, 21
// with 512, 30 with 1024 pairs); a large one gains from fuller chunks (2^24
// pairs: 1,092, 837 and 805 us with 512, 1024 and 2048; 2^20: 81, 66 and 68).
// Up to 4 words per mask eight waves per SIMD fit the registers, and only
// 512-pair tiles leave the LDS for them (2^24 pairs of 100 bases: 475, 563 and
// 774 us).
inline uint32_t mixed_auto_tile(uint64_t n_pairs, uint32_t wmax)
{
    if (wmax <= 4)
        return 512u;
    return n_pairs <= (1u << 17) ? 256u : n_pairs < (1u << 19) ? 512u
         : n_pairs < (1u << 22) ? 1024u : 2048u;
}

// Lanes per pair (log2) of those tiles: 60,001 pairs 17.8 -> 15.2 us with two
// lanes, 131,072 pairs 25.9 -> 21.3 (17.8 and 23.7 with four).
inline uint32_t mixed_auto_lanes(uint64_t n_pairs, uint32_t wmax)
{
    return wmax > 4 && n_pairs <= (1u << 17) ? 1u : 0u;
}

// Batches too small for the sort's steps to pay: with 8 or 4 lanes per pair
// the plain kernel takes 8 to 11 us for up to 16,384 mixed pairs, the sorted one
// 14 and more; at 4 words per mask and fewer it needs no lanes for that (65,536
// pairs of 64 to 128 bases: 7.2 against 9.7 us; 262,144: 14.9 against 12.9).  One
// threshold above 31 leaves nothing to sort, and lanes share only the first 31
// shifts (500 bases, e = 200: 30,000 pairs 217 us plain, 394 sorted; 196,608 pairs
// 536 and 677, 262,144 pairs 710 and 680).
inline bool mixed_unsorted(const FilterArgs &a, uint64_t n_pairs, uint32_t wmax)
{
    return n_pairs <= (!a.e_pair && a.e_uniform > 31u ? 3u << 16 : wmax <= 4 ? 1u << 17 : 24576u);
}

// Whether the plain call sorts its pairs first (the ordered form of the mixed
// launch): a threshold per pair makes a wave of neighbours run the largest of
// its thresholds.  4 M pairs, e per pair up to a tenth of the length: 250 bases
// 384 us as they come, 252 sorted; 150 bases 161 and 135; mixed lengths up to
// 300 944 and 206.  At 4 words per mask and fewer the sort costs more than it
// saves where the lengths are equal (128 bases: 115 and 143 us), and under 2^18
// pairs one wave per SIMD runs either way, without the sort's steps before it.
inline bool filter_sorts(bool e_per_pair, uint64_t n_pairs, uint32_t wmax)
{
    return e_per_pair && wmax >= 5 && n_pairs >= (1u << 18);
}

// Pairs per tile of that form.  Enough tiles for every compute unit: 2^18 pairs
// of 250 bases 32, 25, 31 and 56 us with 256, 512, 1024 and 2048; 2^22 pairs 330,
// 262, 249 and 261.
inline uint32_t filter_tile(uint64_t n_pairs) { return n_pairs < (1u << 19) ? 512u : 1024u; }

struct MixedArgs {
    const BatchTable *table;     // table form: the device table; with n_tiles
                                 // set, a host table of at most INLINE_BATCHES
    uint32_t *tile_counter;      // table form: zeroed by the launch sequence
    uint32_t tile;               // pairs per tile (multiple of 256, <= 2048)
    uint32_t ppl;                // 1 or 2
    uint32_t sort_e;             // 0 or 1
    uint32_t blocks;             // table form: persistent workgroups
    uint32_t n_tiles;            // tiles of a host table, else 0
    uint32_t lg;                 // direct form: 2^lg lanes per pair (0 or 1)
};

// A table of few batches, passed as kernel arguments: the launch then waits for
// no copy of its table.  As many as fit beside the kernel's other arguments in
// the 4 KiB that a launch may pass.
constexpr uint32_t INLINE_BATCHES =
    (4096 - sizeof(FilterArgs) - sizeof(MixedArgs) - 2 * sizeof(uint32_t)) /
    (sizeof(FilterArgs) + sizeof(uint32_t));
struct InlineTable {
    uint32_t n_batches;
    uint32_t prefix[INLINE_BATCHES + 1];
    FilterArgs args[INLINE_BATCHES];
};
static_assert(sizeof(FilterArgs) + sizeof(MixedArgs) + sizeof(InlineTable) <= 4096,
              "passed to one launch");

}  // namespace gkd
