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

// The same through one list of the whole batch's pairs, for a batch with one
// threshold (a.e_pair NULL, a.e_uniform <= GK_VERIFY_MAX_E).
struct VerifyScratch {
    uint32_t *list;      // min(n_pairs, 2^30) words
    uint32_t *groups;    // a word per 4096 of those pairs, rounded up
    uint32_t *count;     // one word
};
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

// Whether a batch is listed as a whole.  Where the band's column loop is the
// whole cost, planes in registers and full waves beat the tile form: 2^22 pairs
// of 150 bases at e = 15 148 against 180 us, of 250 at e = 25 518 against 599,
// of 100 at e = 10 85 against 98; at e <= 7 (furthest-reaching points) 63
// against 76 us the other way.  Its four launches take 20 us before any work,
// so small batches stay with one.
inline bool verify_lists(bool e_per_pair, uint32_t e, uint64_t n_pairs)
{
    return !e_per_pair && e >= 8 && e <= GK_VERIFY_MAX_E &&
           n_pairs >= (e >= 16 ? 1u << 17 : e >= 12 ? 1u << 18 : 1u << 19);
}

}  // namespace gkd
