// Launcher of the verification kernels (gk_verify).
#pragma once

#include "gk_args.h"

namespace gkd {

// dist[i] = min(edit distance, e_i + 1) for the pairs with accept[i] ==
// GK_ACCEPT (every pair when accept is NULL); GK_EST_NONE for the others and
// for pairs that cannot be compared or have e_i > GK_VERIFY_MAX_E.  words:
// 32-base words of the longest read.  One launch per 2^30 pairs, no scratch.
hipError_t launch_verify(const FilterArgs &a, const uint8_t *accept, uint16_t *dist,
                         uint32_t words, uint32_t layout, hipStream_t s);

// The same through one list of the whole batch's pairs: of a batch with one
// threshold (a.e_uniform <= GK_VERIFY_MAX_E), or with a threshold per pair, a
// read index per pair and n_reads > 0.
struct VerifyScratch {
    uint32_t *list;      // min(n_pairs, 2^30) words
    uint32_t *groups;    // one threshold: a word per 4096 of those pairs, rounded up
    uint32_t *count;     // one word
    uint32_t *bins;      // a threshold per pair: VERIFY_BIN_WORDS words
    uint32_t *reads;     // the same: n_reads * verify_read_stride(rows) words, 16-byte aligned
};
constexpr uint32_t VERIFY_BIN_WORDS = 3u * 512u * 32u;
inline uint32_t verify_read_stride(uint32_t rows) { return (rows + 3u) & ~3u; }
hipError_t launch_verify_listed(const FilterArgs &a, const uint8_t *accept, uint16_t *dist,
                                uint32_t words, uint32_t layout, const VerifyScratch &x, int cus,
                                hipStream_t s);

// Pairs per workgroup of launch_verify.  Few pairs: tiles for every compute unit
// (65,536 pairs of 100 bases, e = 5: 9 us with 256 pairs, 13 with 1024, 20 with
// 2048); many: fewer partly filled waves (2^22 pairs of mixed lengths with a
// threshold per pair: 818, 434, 262 and 233 us with 256, 512, 1024 and 2048).
inline uint32_t verify_tile(uint64_t n_pairs)
{
    return n_pairs < (1u << 17) ? 256u : n_pairs < (1u << 19) ? 512u
         : n_pairs < (3u << 18) ? 1024u : 2048u;
}

// Whether a batch is listed as a whole.
//
// One threshold of 8 or more: the band's column loop is the whole cost, and
// planes in registers and full waves beat the tile form: 2^22 pairs of 150 bases
// at e = 15 148 against 180 us, of 250 at e = 25 518 against 599, of 100 at e = 10
// 85 against 98.  One threshold up to 7: full waves, however few of the pairs are
// listed: 2^22 pairs of 100 bases at e = 5 57 against 67 us, 2^26 of 250 at e = 7
// 1,742 against 2,351 with a third listed and 620 against 1,096 with a fifteenth.
// The four launches take 20 us before any work, so smaller batches stay with one;
// from 16 on that is up to one tile per compute unit (250 bases, e = 25: 65,536
// pairs 30 us by tile and 36 by list, 98,304 pairs 42 and 36).
//
// A threshold per pair: the list is in order of (words, e) over the batch, which
// takes each read's candidates apart, so the reads are copied row by row first.
// From about 12 candidates per read on that pays at any share listed (13 per
// read, 3 * 2^19 pairs, tile against list: 111 and 91 us with a sixth listed, 90
// and 71 with a twentieth, but 2^20 pairs 71 and 80, 51 and 67; 24 per read, 2^26
// pairs: 2,477 and 2,044), with 7 from 2^24 pairs on (757 and 670 us, 366 and 347;
// 2^22 pairs 218 and 190, 97 and 108), with 3 at none.
inline bool verify_lists(const FilterArgs &a)
{
    if (a.e_pair)
        return a.pair_read && a.n_reads > 0 && a.n_pairs >= (3u << 19) &&
               a.n_pairs / (a.n_pairs >= (1u << 24) ? 7u : 12u) >= a.n_reads;
    const uint32_t e = a.e_uniform;
    return e <= GK_VERIFY_MAX_E && a.n_pairs >= (e >= 16  ? (1u << 16) + 1u
                                                 : e >= 12 ? 1u << 18
                                                 : e >= 8  ? 1u << 19
                                                           : 1u << 22);
}

}  // namespace gkd
