// Verification of filtered pairs: the exact edit distance (unit-cost global
// alignment of the read and its window, the ground truth of Sec. 4.4) that the
// read mapper's verification step computes for the pairs the filter passes
// (Sec. 3.3, Sec. 3.5), capped at e + 1.
//
// One lane computes one pair, by one of two algorithms:
//
// Furthest-reaching points on the diagonals of the dynamic-programming matrix
// (Ukkonen; Myers' O(ND) algorithm), for e <= 7: F(d, k) is the number of read
// bases consumed by the furthest path with at most d edits that ends on
// diagonal k = window position - read position,
//   F(d, k) = slide(max(F(d-1, k) + 1, F(d-1, k+1) + 1, F(d-1, k-1))),
// where slide follows matches along the diagonal, and the distance is the
// least d with F(d, 0) = m.  A path on diagonal k after d edits needs |k| more
// to come back, so with a cap of e only |k| <= min(d, e - d) is computed: 18
// points for e = 5, of about 25 instructions each, where a band column takes
// 22 (16 with two pairs to a word) for each of the read's bases.  A slide
// compares 32 bases at a time: the pair's bit-planes lie in LDS, one column
// per lane, two neighbouring words of read and window give the 32 bases from
// any position with funnel shifts, and the first mismatch is a find-first-bit.
//
// The banded bit-vector algorithm above that (banded_distance): one pass over
// the window's bases whatever e is, in a 32-bit word up to e = 15 and a 64-bit
// one up to 31.  Its points overtake it in number from e = 10 on (61), and with
// LDS latency in each they do from e = 8 (100 bases, e = 10, 2^22 pairs: 106 us
// against 98).
//
// Tile form (k_verify_tile): a workgroup takes a tile of T consecutive pairs,
// lists the ones to verify in LDS, counting-sorted by (words of the read, e) so
// that a wave's lanes load alike and run alike, and its waves take 64 of the
// list at a time, the longest first.  Distances replace the pairs' entries in
// LDS and go to memory in pair order.  One launch; listing the whole batch
// first takes four to six (1,000 pairs of 100 bases at e = 5: 22 -> 9 us; 2^20
// pairs of mixed lengths and thresholds 113 -> 72, 1,000 pairs 98 -> 39).
//
// List form: large batches whose tiles would leave waves partly filled go through
// one list of all their pairs (verify_lists; 2^22 pairs of 100 bases at e = 5 62
// us, 70 by tile).
#include <algorithm>

#include "gk_pair.h"
#include "gk_verify.h"

namespace gkd {
namespace {

constexpr uint32_t VBINS = 16 * 32;          // words 1..16, e 0..31
constexpr uint32_t FURTHEST_MAX_E = 7;
constexpr uint32_t NOT_LISTED = 0xFFFFu;     // = GK_EST_NONE

struct VerifyLds {
    uint32_t hist[VBINS];
    uint32_t total;
    uint32_t next;
    uint32_t pad_[2];
};

// Plane words of one wave: column `lane`, word w at [w * 64 + lane], the read's
// in the first words + 1 rows, the window's in the next.  (The last row of each
// only fills the funnel at a read's end.)
__host__ __device__ inline uint32_t wave_planes(uint32_t words) { return 2u * (words + 1u) * 64u; }

size_t verify_lds_bytes(uint32_t words, uint32_t tile)
{
    return sizeof(VerifyLds) + 4u * wave_planes(words) * sizeof(uint2) + 2u * tile * 2u;
}

// Tile of a batch: verify_tile's, and from 2^22 pairs on up to 8192 while as many
// workgroups fit a compute unit.  Longer lists have fewer waves of mixed lengths
// and thresholds: 2^24 pairs of 64 to 300 bases with a threshold per pair, a
// third listed, 1,123, 981 and 996 us with 2048, 4096 and 8192 pairs, a seventh
// listed 730, 622 and 602 (two workgroups each); but 2^24 of 250 bases 1,155,
// 1,442 and 1,617 (three, two and two).
uint32_t tile_of(uint64_t n_pairs, uint32_t words)
{
    const size_t lds = 160u * 1024u;
    uint32_t tile = verify_tile(n_pairs);
    if (n_pairs >= (1u << 22)) {
        const size_t fit = lds / verify_lds_bytes(words, tile);
        while (tile < 8192u && lds / verify_lds_bytes(words, 2u * tile) == fit)
            tile *= 2u;
    }
    return tile;
}

// A lane's column of its wave's planes: the read's words at read[w * 64], the
// window's at text[w * 64].
struct Column {
    uint2 *read, *text;
};

__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    return __builtin_amdgcn_readfirstlane(v);
}

// Bit b: read base i + b differs from window base j + b (both inside the planes).
__device__ __forceinline__ uint32_t differ32(const Column &col, int i, int j)
{
    const uint2 *r = col.read + ((uint32_t)i >> 5) * 64u;
    const uint2 *g = col.text + ((uint32_t)j >> 5) * 64u;
    const uint2 r0 = r[0], r1 = r[64], g0 = g[0], g1 = g[64];
    // the funnel takes the shift modulo 32
    const uint32_t rh = funnel(r1.x, r0.x, (uint32_t)i), rl = funnel(r1.y, r0.y, (uint32_t)i);
    const uint32_t gh = funnel(g1.x, g0.x, (uint32_t)j), gl = funnel(g1.y, g0.y, (uint32_t)j);
    return (rh ^ gh) | (rl ^ gl);
}

__device__ __forceinline__ int first_of(uint32_t x) { return x ? __builtin_ctz(x) : 32; }

// Matches from read base i on diagonal k, at most `left` (0 or more), after
// the first n (the first 32 compared).
__device__ __forceinline__ int slide_on(const Column &col, int i, int k, int left, int n)
{
    int t = n;
    while (n == 32 && t < left) {
        n = first_of(differ32(col, i + t, i + t + k));
        t += n;
    }
    return t < left ? t : left;
}

__device__ __forceinline__ int slide(const Column &col, int i, int k, int left)
{
    const int at = left > 0 ? i : 0;         // (any place inside the planes will do)
    return slide_on(col, i, k, left,
                          first_of(differ32(col, at, left > 0 ? i + k : 0)));
}

// Diagonals k and -k, then outwards, of one more edit: F[q + K + 1] = F(d, q)
// from F(d-1, .) in place, up = F(d-1, k-1), down = F(d-1, 1-k).  The two
// slides' first 32 bases are compared with both pairs of loads in flight.
template <int K, int k>
__device__ __forceinline__ void outwards(const Column &col, int m, int reach, int (&F)[2 * K + 3],
                                         int up, int down)
{
    if constexpr (k <= K) {
        if (k <= reach) {
            const int hp = F[K + 1 + k], op = F[K + 2 + k];
            const int hn = F[K + 1 - k], on = F[K - k];
            int ip = (hp > op ? hp : op) + 1;
            ip = ip > up ? ip : up;
            ip = ip < m - k ? ip : m - k;
            int in = (hn > down ? hn : down) + 1;
            in = in > on ? in : on;
            in = in < m ? in : m;
            const int lp = m - k - ip, ln = m - in;
            const uint32_t xp = differ32(col, lp > 0 ? ip : 0, lp > 0 ? ip + k : 0);
            const uint32_t xn = differ32(col, ln > 0 ? in : k, ln > 0 ? in - k : 0);
            F[K + 1 + k] = ip + slide_on(col, ip, k, lp, first_of(xp));
            F[K + 1 - k] = in + slide_on(col, in, -k, ln, first_of(xn));
            outwards<K, k + 1>(col, m, reach, F, hp, hn);
        }
    }
}

// min(distance, e + 1) of the lane's pair by furthest-reaching points;
// E >= every lane's e, E / 2 <= K.  Lanes without a pair pass m = 0.
template <int K>
__device__ __forceinline__ uint32_t furthest_distance(const Column &col, int m, uint32_t e,
                                                      uint32_t E)
{
    int F[2 * K + 3];
#pragma unroll
    for (int q = 0; q < 2 * K + 3; ++q)
        F[q] = -1000;
    F[K + 1] = slide(col, 0, 0, m);
    uint32_t dist = F[K + 1] >= m ? 0u : e + 1u;
#pragma unroll 1
    for (uint32_t d = 1; d <= E; ++d) {
        if (__ballot(dist > e && d <= e) == 0ull)
            break;
        const int here = F[K + 1];
        int i = (here > F[K + 2] ? here : F[K + 2]) + 1;
        i = i > F[K] ? i : F[K];
        i = i < m ? i : m;
        F[K + 1] = i + slide(col, i, 0, m - i);
        // (m opaque: m - k of every diagonal is not kept in a register)
        asm volatile("" : "+v"(m));
        outwards<K, 1>(col, m, (int)(d < E - d ? d : E - d), F, here, here);
        if (dist > e && d <= e && F[K + 1] >= m)
            dist = d;
    }
    return dist;
}

// A 64-bit band word kept as two 32-bit halves, so that chains of logic
// operations on it map onto 3-input logic instructions per half (whole 64-bit
// values get split into halves only after that combining is done).
struct B64 {
    uint32_t lo, hi;
};
__device__ __forceinline__ B64 operator&(B64 a, B64 b) { return {a.lo & b.lo, a.hi & b.hi}; }
__device__ __forceinline__ B64 operator|(B64 a, B64 b) { return {a.lo | b.lo, a.hi | b.hi}; }
__device__ __forceinline__ B64 operator^(B64 a, B64 b) { return {a.lo ^ b.lo, a.hi ^ b.hi}; }
__device__ __forceinline__ B64 operator~(B64 a) { return {~a.lo, ~a.hi}; }
__device__ __forceinline__ B64 operator+(B64 a, B64 b)
{
    const uint64_t s = (((uint64_t)a.hi << 32) | a.lo) + (((uint64_t)b.hi << 32) | b.lo);
    return {(uint32_t)s, (uint32_t)(s >> 32)};
}

template <typename T> __device__ __forceinline__ T from64(uint64_t v);
template <> __device__ __forceinline__ uint32_t from64<uint32_t>(uint64_t v) { return (uint32_t)v; }
template <> __device__ __forceinline__ B64 from64<B64>(uint64_t v)
{
    return {(uint32_t)v, (uint32_t)(v >> 32)};
}

// all-zero / all-one mask of one text code bit
template <typename T> __device__ __forceinline__ T broadcast(uint32_t m);
template <> __device__ __forceinline__ uint32_t broadcast<uint32_t>(uint32_t m) { return m; }
template <> __device__ __forceinline__ B64 broadcast<B64>(uint32_t m) { return {m, m}; }

__device__ __forceinline__ uint32_t shr1(uint32_t x) { return x >> 1; }
__device__ __forceinline__ B64 shr1(B64 x) { return {funnel(x.hi, x.lo, 1), x.hi >> 1}; }

// bit e of x; e <= 31 in both widths (the wide band serves 16 <= e <= 31)
__device__ __forceinline__ uint32_t bit_at(uint32_t x, uint32_t e) { return (x >> e) & 1u; }
__device__ __forceinline__ uint32_t bit_at(B64 x, uint32_t e) { return (x.lo >> e) & 1u; }

// One column step of the banded edit distance.  bh, bl: the band's read-plane
// bits (bit k = read base j - e + k - 1, 0-based, for text column j); th, tl:
// the text base's code bits as all-zero / all-one masks.  vp, vn come in
// already slid down one row into this column's band (bit 2e, the new bottom
// row, steps +1) and leave slid into the next column's: the slide's shift
// right cancels the shift left of the horizontal deltas, so the next column's
// vertical deltas at band row k read the horizontal deltas of row k and the
// XV bit of row k + 1 directly.  Bits above 2e may hold anything in eq, xh, ph
// and mh: carries and shifts only move information upward there, and the
// masks keep them out of vp and vn.
template <typename T>
__device__ __forceinline__ T band_column(T eq, T top, T keep, T &vp, T &vn)
{
    const T xh = (((eq & vp) + vp) ^ vp) | eq;
    const T diag = xh | vn;              // bit e: the diagonal did not step +1
    // Horizontal deltas +1 / -1 of the band rows.  The row above the band
    // (+1) would only enter bit 0 of this column's new vertical deltas, which
    // the slide drops.
    const T ph = vn | ~(xh | vp);
    const T mh = vp & xh;
    const T xv1 = shr1(eq | vn);         // XV of the next column's band rows
    vp = ((mh | ~(xv1 | ph)) & keep) | top;
    vn = ph & xv1 & keep;
    return diag;
}

template <typename T>
__device__ __forceinline__ void band_step(T bh, T bl, T th, T tl, T top, T keep, uint32_t e,
                                          T &vp, T &vn, uint32_t &flat)
{
    const T eq = ~((bh ^ th) | (bl ^ tl));
    flat += bit_at(band_column(eq, top, keep, vp, vn), e);
}

// 32 (T = uint32_t) or 64 (T = B64) bits of [a | b | c] from bit s of a.
template <typename T>
__device__ __forceinline__ T bits_from(uint32_t a, uint32_t b, uint32_t c, uint32_t s)
{
    const uint32_t lo = funnel(b, a, s);
    if constexpr (sizeof(T) == 4)
        return lo;
    else
        return B64{lo, funnel(c, b, s)};
}

// min(distance, e + 1) of the lane's pair by the band of the 2E+1 diagonals
// |i - j| <= E, E >= every lane's e (E <= 15 in 32 bits, E <= 31 in 64); one
// pass over the window's bases, whatever the distance.  The vertical
// differences of the band are one word of 2E+1 bits; per text column the band
// slides down one row and the column step of Myers' bit-vector algorithm (in
// Hyyro's formulation) updates it.  Boundary choices:
//   - rows above row 0 are virtual with D[i][j] = j - i, which keeps
//     D[0][j] = j and satisfies the recurrence whatever they match, so the
//     band slides from the first column on;
//   - the cell above the band takes D[i][j-1] + 1 and the cell entering at
//     the band's bottom takes D[i-1][j] + 1: both bound the true values from
//     above, so every band value is an upper bound, and it is exact along any
//     path of cost <= E;
//   - rows below the read end never influence row m.
// The diagonal cell D[j][j] is tracked through the band's diagonal zero-delta
// bit, and D[m][m] is the result.
//
// Read bases are taken from [32 zero bits | plane words 0..words-1 | zeros]:
// for text column j = 32 blk + c + 1 the band starts at extended bit
// 32 blk + c + 32 - E, which lies in extended word blk (read word blk - 1)
// while c < E and in word blk + 1 (read word blk) from c = E on; the column
// loop is split there so each part reads fixed words.
template <typename T>
__device__ __forceinline__ uint32_t banded_distance(const Column &col, uint32_t m, uint32_t e,
                                                    uint32_t E, uint32_t words)
{
    const uint64_t top64 = 1ull << (2 * E);        // band row 2E: enters each column
    const uint64_t keep64 = top64 - 1;             // band rows 0 .. 2E-1 after a slide
    const uint64_t vn0 = (2ull << E) - 1;          // column 0: rows -E..0 step -1,
    const uint64_t vp0 = (top64 | keep64) & ~vn0;  //           rows 1..E step +1
    const T top = from64<T>(top64), keep = from64<T>(keep64);
    T vp = from64<T>(((vp0 >> 1) & keep64) | top64);   // slid into column 1's band
    T vn = from64<T>((vn0 >> 1) & keep64);
    uint32_t flat = 0;                             // columns j where D[j][j] = D[j-1][j-1]
    uint2 r0 = make_uint2(0u, 0u), r1 = col.read[0], r2 = col.read[64];
#pragma unroll 1
    for (uint32_t blk = 0; blk < words; ++blk) {
        const uint2 r3 = blk + 2u <= words ? col.read[(blk + 2u) * 64u] : make_uint2(0u, 0u);
        const uint2 text = col.text[blk * 64u];
        const int cols = (int)m - (int)(32u * blk) < 32 ? (int)m - (int)(32u * blk) : 32;
        const int split = (int)E < cols ? (int)E : cols;
        for (int c = 0; c < split; ++c) {          // band starts in read word blk - 1
            const uint32_t s = (uint32_t)c + 32u - E;
            band_step<T>(bits_from<T>(r0.x, r1.x, r2.x, s), bits_from<T>(r0.y, r1.y, r2.y, s),
                         broadcast<T>(__builtin_amdgcn_sbfe(text.x, c, 1)),
                         broadcast<T>(__builtin_amdgcn_sbfe(text.y, c, 1)), top, keep, E, vp, vn,
                         flat);
        }
        for (int c = (int)E; c < cols; ++c) {      // band starts in read word blk
            const uint32_t s = (uint32_t)c - E;
            band_step<T>(bits_from<T>(r1.x, r2.x, r3.x, s), bits_from<T>(r1.y, r2.y, r3.y, s),
                         broadcast<T>(__builtin_amdgcn_sbfe(text.x, c, 1)),
                         broadcast<T>(__builtin_amdgcn_sbfe(text.y, c, 1)), top, keep, E, vp, vn,
                         flat);
        }
        r0 = r1;
        r1 = r2;
        r2 = r3;
    }
    const uint32_t score = m - flat;               // D[m][m]: each diagonal step is 0 or +1
    return score < e + 1u ? score : e + 1u;
}

// A wave whose pairs share the length keeps the column loops' bounds scalar.
template <typename T>
__device__ __forceinline__ uint32_t banded(const Column &col, uint32_t m, bool have, uint32_t e,
                                           uint32_t E, uint32_t words)
{
    const uint32_t m0 = wave_max(have ? m : 0u);
    if (__ballot(have && m != m0) == 0ull)
        return banded_distance<T>(col, m0, e, E, words);
    return banded_distance<T>(col, m, e, E, words);
}

// Loads one pair and puts its planes into the lane's column.  Returns whether
// the pair can be compared.
template <int W, int L, bool ROWWISE>
__device__ __forceinline__ bool load_planes(const FilterArgs &a, const PairIdx &p, const Column &col)
{
    PairData<W> d;
    load_data<W, ROWWISE>(a, p, d);
    uint32_t m;
    const bool ok = pair_gate<W>(a, p, d, m) == PAIR_OK;
    uint32_t gh[W], gl[W], rh[W], rl[W];
    pair_planes<W, L>(p, d, gh, gl, rh, rl);
#pragma unroll
    for (int w = 0; w < W; ++w) {
        gh[w] &= ones_below((int)m - 32 * w);
        gl[w] &= ones_below((int)m - 32 * w);
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        col.read[w * 64] = make_uint2(rh[w], rl[w]);
        col.text[w * 64] = make_uint2(gh[w], gl[w]);
    }
    col.read[W * 64] = make_uint2(0u, 0u);
    col.text[W * 64] = make_uint2(0u, 0u);
    return ok;
}

template <int WMAX, int L, bool ROWWISE>
__device__ __forceinline__ bool load_planes_w(const FilterArgs &a, const PairIdx &p, uint32_t w,
                                              const Column &col)
{
#define GK_CASE(N)                                                                 \
    case N:                                                                        \
        if (N <= WMAX)                                                             \
            return load_planes<(N <= WMAX ? N : 1), L, ROWWISE>(a, p, col);  \
        break;
    switch (w) {
        GK_CASE(1) GK_CASE(2) GK_CASE(3) GK_CASE(4) GK_CASE(5) GK_CASE(6) GK_CASE(7) GK_CASE(8)
        GK_CASE(9) GK_CASE(10) GK_CASE(11) GK_CASE(12) GK_CASE(13) GK_CASE(14) GK_CASE(15)
        GK_CASE(16)
    default:
        break;
    }
#undef GK_CASE
    return false;
}

// Distances of a wave's pairs, one per lane: len the read's length where the
// lane has a pair with p.e <= GK_VERIFY_MAX_E, else 0 (p is then any pair whose
// loads may be issued).
template <int WMAX, int L, bool ROWWISE = false>
__device__ __forceinline__ uint32_t wave_distances(const FilterArgs &a, const PairIdx &p,
                                                   uint32_t len, const Column &col)
{
    FilterArgs ac = a;         // (nor the row addresses of every width)
    asm volatile("" : "+s"(ac.pitch), "+s"(ac.rows), "+s"(ac.max_read_len));
    const uint32_t e = len != 0u ? p.e : 0u;
    const uint32_t w = wave_max((len + 31u) / 32u);
    const uint32_t E = wave_max(e);
    const bool ok = load_planes_w<WMAX, L, ROWWISE>(ac, p, w, col) && len != 0u;
    const uint32_t m = ok ? len : 0u;
    uint32_t d;
    if (E <= FURTHEST_MAX_E)
        d = furthest_distance<FURTHEST_MAX_E / 2>(col, (int)m, e, E);
    else if (E <= 15u)
        d = banded<uint32_t>(col, m, ok, e, E, w);
    else
        d = banded<B64>(col, m, ok, e, E, w);
    return ok ? d : GK_EST_NONE;
}

// Bin of an entry: words of the read, e.
__device__ __forceinline__ uint32_t entry_key(uint32_t en)
{
    return (((en & 0x3FFu) + 31u) / 32u - 1u) * 32u + (en >> 10);
}

template <int WMAX, int L>
__global__ __launch_bounds__(256) void k_verify_tile(FilterArgs a, const uint8_t *accept,
                                                     uint16_t *dist, uint32_t tile,
                                                     uint32_t words)
{
    extern __shared__ uint32_t lds_raw[];
    VerifyLds &s = *reinterpret_cast<VerifyLds *>(lds_raw);
    uint2 *planes = reinterpret_cast<uint2 *>(lds_raw + sizeof(VerifyLds) / 4);
    uint16_t *entry = reinterpret_cast<uint16_t *>(planes + 4u * wave_planes(words));
    uint16_t *list = entry + tile;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t n = (uint32_t)a.n_pairs;
    const uint32_t base = blockIdx.x * tile;

    for (uint32_t b = tid; b < VBINS; b += 256)
        s.hist[b] = 0;
    __syncthreads();

    // 1. list the pairs to verify: entry = length | e << 10, key = words, e
    for (uint32_t j0 = tid; j0 < tile; j0 += 1024) {
        uint32_t on[4], r[4], e[4], m[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = base + j0 + 256u * q, c = i < n ? i : n - 1u;
            on[q] = accept ? (accept[c] == GK_ACCEPT) : 1u;
            r[q] = a.pair_read ? a.pair_read[c] : c;
            e[q] = a.e_pair ? (uint32_t)a.e_pair[c] : a.e_uniform;
            on[q] = on[q] && i < n && e[q] <= GK_VERIFY_MAX_E && r[q] < a.n_reads;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            m[q] = a.read_len[on[q] ? r[q] : 0u];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t j = j0 + 256u * q;
            if (j >= tile)
                break;
            uint32_t en = NOT_LISTED;
            if (on[q] && m[q] != 0u && m[q] <= a.max_read_len) {
                en = m[q] | (e[q] << 10);
                atomicAdd(&s.hist[entry_key(en)], 1u);
            }
            entry[j] = (uint16_t)en;
        }
    }
    __syncthreads();

    // 2. exclusive prefix over the bins
    if (tid < 64) {
        uint32_t local[8], sum = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            local[q] = s.hist[tid * 8 + q];
            sum += local[q];
        }
        uint32_t run = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(run, o, 64);
            if (lane >= (uint32_t)o)
                run += v;
        }
        if (tid == 63) {
            s.total = run;
            s.next = 0;
        }
        run -= sum;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            s.hist[tid * 8 + q] = run;
            run += local[q];
        }
    }
    __syncthreads();

    // 3. slots in key order
    for (uint32_t j = tid; j < tile; j += 256) {
        const uint32_t en = entry[j];
        if (en != NOT_LISTED)
            list[atomicAdd(&s.hist[entry_key(en)], 1u)] = (uint16_t)j;
    }
    __syncthreads();

    // 4. waves take 64 at a time from the end of the list
    const uint32_t total = s.total;
    Column col;
    col.read = planes + (tid >> 6) * wave_planes(words) + lane;
    col.text = col.read + (words + 1u) * 64u;
    while (true) {
        uint32_t c = 0;
        if (lane == 0)
            c = atomicAdd(&s.next, 64u);
        c = __builtin_amdgcn_readfirstlane(c);
        if (c >= total)
            break;
        const uint32_t at = c + lane;
        const bool have = at < total;
        // Lanes past the list's end load the wave's first pair, whose loads are
        // in flight anyway, and take no part: its entry may hold a result by now.
        const uint32_t slot = list[have ? total - 1u - at : total - 1u - c];
        const uint32_t en = have ? entry[slot] : 0u;
        PairIdx p = load_idx(a, base + slot);
        p.e = en >> 10;
        const uint32_t d = wave_distances<WMAX, L>(a, p, en & 0x3FFu, col);
        if (have)
            entry[slot] = (uint16_t)d;
    }
    __syncthreads();

    // 5. distances in pair order
    for (uint32_t j = tid; j < tile; j += 256)
        if (base + j < n)
            dist[base + j] = entry[j];
}

template <int WMAX, int L>
hipError_t tile_wl(const FilterArgs &a, const uint8_t *accept, uint16_t *dist, uint32_t words,
                     uint32_t tile, hipStream_t s)
{
    const uint64_t CHUNK = 1ull << 30;
    for (uint64_t first = 0; first < a.n_pairs; first += CHUNK) {
        FilterArgs c = a;
        const uint64_t n = a.n_pairs - first < CHUNK ? a.n_pairs - first : CHUNK;
        c.n_pairs = n;
        c.pair_read = a.pair_read ? a.pair_read + first : nullptr;
        if (!a.pair_read && first > 0)
            c.n_reads = 0;   // pair i uses read i < n_reads < 2^30: none here
        c.cand_pos = a.cand_pos + first;
        c.e_pair = a.e_pair ? a.e_pair + first : nullptr;
        hipLaunchKernelGGL((k_verify_tile<WMAX, L>), dim3((uint32_t)((n + tile - 1) / tile)), dim3(256),
                           verify_lds_bytes(words, tile), s, c, accept ? accept + first : nullptr,
                           dist + first, tile, words);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <int L>
hipError_t tile_l(const FilterArgs &a, const uint8_t *accept, uint16_t *dist, uint32_t words,
                  uint32_t tile, hipStream_t s)
{
    if (words <= 4)
        return tile_wl<4, L>(a, accept, dist, words, tile, s);
    if (words <= 8)
        return tile_wl<8, L>(a, accept, dist, words, tile, s);
    if (words <= 10)
        return tile_wl<10, L>(a, accept, dist, words, tile, s);
    return tile_wl<16, L>(a, accept, dist, words, tile, s);
}

// ---- one list over the whole batch ---------------------------------------
//
// Large batches (verify_lists).  Under one threshold of 8 and more the band's
// column loop is the whole cost, and it runs fastest with the planes in
// registers (no LDS but the tile form's, whose columns leave 3 waves per SIMD at
// 8 words) and full waves from one list; smaller thresholds and batches with a
// threshold per pair take the tile form's algorithms in full waves.

// Read bases are taken from [32 zero bits | plane words 0..W-1 | zeros]: for
// text column j = 32 blk + c + 1 the band starts at extended bit
// 32 blk + c + 32 - e, which lies in extended word blk (read word blk - 1)
// while c < e and in word blk + 1 (read word blk) from c = e on; the column
// loop is split there so each part reads fixed words.
template <int W, typename T>
__device__ __forceinline__ uint32_t band_distance(const uint32_t (&rh)[W], const uint32_t (&rl)[W],
                                                  const uint32_t (&gh)[W], const uint32_t (&gl)[W],
                                                  uint32_t m, uint32_t e)
{
    const uint64_t top64 = 1ull << (2 * e);        // band row 2e: enters each column
    const uint64_t keep64 = top64 - 1;             // band rows 0 .. 2e-1 after a slide
    const uint64_t vn0 = (2ull << e) - 1;          // column 0: rows -e..0 step -1,
    const uint64_t vp0 = (top64 | keep64) & ~vn0;  //           rows 1..e step +1
    const T top = from64<T>(top64), keep = from64<T>(keep64);
    T vp = from64<T>(((vp0 >> 1) & keep64) | top64);   // slid into column 1's band
    T vn = from64<T>((vn0 >> 1) & keep64);
    uint32_t flat = 0;                             // columns j where D[j][j] = D[j-1][j-1]
#pragma unroll
    for (int blk = 0; blk < W; ++blk) {
        const uint32_t h0 = blk >= 1 ? rh[blk - 1] : 0u, l0 = blk >= 1 ? rl[blk - 1] : 0u;
        const uint32_t h1 = rh[blk], l1 = rl[blk];
        const uint32_t h2 = blk + 1 < W ? rh[blk + 1] : 0u, l2 = blk + 1 < W ? rl[blk + 1] : 0u;
        const uint32_t h3 = blk + 2 < W ? rh[blk + 2] : 0u, l3 = blk + 2 < W ? rl[blk + 2] : 0u;
        const int cols = (int)m - 32 * blk < 32 ? (int)m - 32 * blk : 32;
        const int split = (int)e < cols ? (int)e : cols;
        const uint32_t th_w = gh[blk], tl_w = gl[blk];
        for (int c = 0; c < split; ++c) {          // band starts in read word blk - 1
            const uint32_t s = (uint32_t)c + 32u - e;
            band_step<T>(bits_from<T>(h0, h1, h2, s), bits_from<T>(l0, l1, l2, s),
                         broadcast<T>(__builtin_amdgcn_sbfe(th_w, c, 1)),
                         broadcast<T>(__builtin_amdgcn_sbfe(tl_w, c, 1)), top, keep, e, vp, vn,
                         flat);
        }
        for (int c = split; c < cols; ++c) {       // band starts in read word blk
            const uint32_t s = (uint32_t)c - e;
            band_step<T>(bits_from<T>(h1, h2, h3, s), bits_from<T>(l1, l2, l3, s),
                         broadcast<T>(__builtin_amdgcn_sbfe(th_w, c, 1)),
                         broadcast<T>(__builtin_amdgcn_sbfe(tl_w, c, 1)), top, keep, e, vp, vn,
                         flat);
        }
    }
    const uint32_t score = m - flat;               // D[m][m]: each diagonal step is 0 or +1
    return score < e + 1u ? score : e + 1u;
}

// Distance of one pair that passed the gate under the batch's one threshold.
// When every active lane has the same length (always so for one read length)
// the band's trip counts come from scalar registers.
template <int W, int L>
__device__ __forceinline__ uint32_t verify_pair(const PairIdx &p, const PairData<W> &d,
                                                uint32_t m, uint32_t e)
{
    uint32_t gh[W], gl[W], rh[W], rl[W];
    pair_planes<W, L>(p, d, gh, gl, rh, rl);
#pragma unroll
    for (int w = 0; w < W; ++w) {
        gh[w] &= ones_below((int)m - 32 * w);
        gl[w] &= ones_below((int)m - 32 * w);
    }
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(m);
    if (__ballot(m != m0) == 0ull)
        return e <= 15u ? band_distance<W, uint32_t>(rh, rl, gh, gl, m0, e)
                        : band_distance<W, B64>(rh, rl, gh, gl, m0, e);
    return e <= 15u ? band_distance<W, uint32_t>(rh, rl, gh, gl, m, e)
                    : band_distance<W, B64>(rh, rl, gh, gl, m, e);
}

// Persistent over the list, one pair per lane.
template <int W, int L>
__global__ __launch_bounds__(256) void k_verify_list(FilterArgs a, const uint32_t *list,
                                                     const uint32_t *count, uint16_t *dist)
{
    const uint32_t n = *count;
    const uint32_t stride = gridDim.x * 256u;
    for (uint32_t t = blockIdx.x * 256u + threadIdx.x; t < n; t += stride) {
        const uint32_t i = list[t];
        const PairIdx p = load_idx(a, i);
        PairData<W> d;
        load_data<W>(a, p, d);
        uint32_t m, out = GK_EST_NONE;
        if (pair_gate<W>(a, p, d, m) == PAIR_OK)
            out = verify_pair<W, L>(p, d, m, a.e_uniform);
        dist[i] = (uint16_t)out;
    }
}

// Listing the pairs to verify (accept[i] == GK_ACCEPT, or every pair when
// accept is NULL) without a contended counter: a workgroup covers 4096
// consecutive pairs, 16 per lane (one 16-byte load of accept when VEC);
// k_select_count stores each workgroup's count, k_select_scan turns the
// counts into offsets (and the total into *count), k_select_write puts each
// workgroup's pairs at its offset through LDS: in pair order when they all
// have one read length, else ordered by it, so that the waves of the verify
// kernel see one length (its fast path needs it).  VEC needs accept and dist
// aligned to 16 bytes; the host checks.
constexpr uint32_t SEL_PER_LANE = 16u, SEL_PER_GROUP = 256u * SEL_PER_LANE;

// Bit j of the result: pair i0 + j is listed.  With fill, the 16 dist entries
// are set to GK_EST_NONE first (the listed ones are overwritten later).
template <bool VEC>
__device__ __forceinline__ uint32_t select_bits(const uint8_t *accept, uint32_t n, uint32_t i0,
                                                uint16_t *dist, bool fill)
{
    const uint32_t valid = i0 < n ? (n - i0 < SEL_PER_LANE ? n - i0 : SEL_PER_LANE) : 0u;
    uint32_t sel = 0;
    if (accept == nullptr) {
        sel = valid == SEL_PER_LANE ? 0xFFFFu : ((1u << valid) - 1u);
    } else if (VEC && valid == SEL_PER_LANE) {
        const uint4 v = *reinterpret_cast<const uint4 *>(accept + i0);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                sel |= (((w[q] >> (8 * b)) & 0xFFu) == GK_ACCEPT ? 1u : 0u) << (4 * q + b);
        if (fill) {
            const uint4 none = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            reinterpret_cast<uint4 *>(dist + i0)[0] = none;
            reinterpret_cast<uint4 *>(dist + i0)[1] = none;
        }
    } else {
        for (uint32_t j = 0; j < valid; ++j) {
            sel |= (accept[i0 + j] == GK_ACCEPT ? 1u : 0u) << j;
            if (fill)
                dist[i0 + j] = (uint16_t)GK_EST_NONE;
        }
    }
    return sel;
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_select_count(const uint8_t *accept, uint32_t n,
                                                      uint32_t *group_count, uint16_t *dist)
{
    __shared__ uint32_t wave_sum[4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t i0 = blockIdx.x * SEL_PER_GROUP + threadIdx.x * SEL_PER_LANE;
    uint32_t c = (uint32_t)__popc(select_bits<VEC>(accept, n, i0, dist, true));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        c += __shfl_xor(c, o, 64);
    if (lane == 0u)
        wave_sum[wave] = c;
    __syncthreads();
    if (threadIdx.x == 0u)
        group_count[blockIdx.x] = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
}

// One workgroup of 1024 lanes: exclusive prefix sums of groups (<= 2^18)
// counts in place, the total into *count.
__global__ __launch_bounds__(1024) void k_select_scan(uint32_t *group_count, uint32_t groups,
                                                      uint32_t *count)
{
    __shared__ uint32_t wave_sum[16];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t per = (groups + 1023u) / 1024u;
    const uint32_t lo = threadIdx.x * per;
    const uint32_t hi = lo + per < groups ? lo + per : groups;
    uint32_t sum = 0;
    for (uint32_t i = lo; i < hi; ++i)
        sum += group_count[i];
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o)
            incl += t;
    }
    if (lane == 63u)
        wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w)
        before += wave_sum[w];
    uint32_t run = before + incl - sum;
    for (uint32_t i = lo; i < hi; ++i) {
        const uint32_t v = group_count[i];
        group_count[i] = run;
        run += v;
    }
    if (threadIdx.x == 1023u) {
        count[0] = before + incl;
    }
}

// Sort keys of the 16 pairs i0 .. i0 + 15 a lane lists (bit j of sel): the
// read length when a pair can be compared at it (1..max_read_len), else 0 (it
// fails the gate).  With no pair-to-read map the 16 lengths are consecutive and
// come in two 16-byte loads when aligned.
__device__ __forceinline__ void length_keys(const FilterArgs &a, uint32_t i0, uint32_t sel,
                                            uint32_t (&key)[SEL_PER_LANE])
{
    if (a.pair_read == nullptr && i0 + SEL_PER_LANE <= a.n_reads &&
        ((uintptr_t)(a.read_len + i0) & 15u) == 0u) {
        const uint4 v0 = *reinterpret_cast<const uint4 *>(a.read_len + i0);
        const uint4 v1 = *reinterpret_cast<const uint4 *>(a.read_len + i0 + 8);
        const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
            key[j] = (w[j >> 1] >> (16u * (j & 1u))) & 0xFFFFu;
    } else if (a.pair_read != nullptr && sel != 0u && i0 + SEL_PER_LANE <= a.n_pairs &&
               ((uintptr_t)(a.pair_read + i0) & 15u) == 0u) {
        // the 16 read indices in four 16-byte loads (one 64-byte span), the
        // lengths of the listed pairs only
        uint32_t r[SEL_PER_LANE];
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const uint4 v = *reinterpret_cast<const uint4 *>(a.pair_read + i0 + 4u * q);
            r[4u * q] = v.x;
            r[4u * q + 1u] = v.y;
            r[4u * q + 2u] = v.z;
            r[4u * q + 3u] = v.w;
        }
#pragma unroll
        for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
            key[j] = (sel & (1u << j)) && r[j] < a.n_reads ? (uint32_t)a.read_len[r[j]] : 0u;
    } else {
#pragma unroll
        for (uint32_t j = 0; j < SEL_PER_LANE; ++j) {
            key[j] = 0u;
            if (sel & (1u << j)) {
                const uint32_t r = a.pair_read ? a.pair_read[i0 + j] : i0 + j;
                key[j] = r < a.n_reads ? (uint32_t)a.read_len[r] : 0u;
            }
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        key[j] = key[j] <= a.max_read_len ? key[j] : 0u;
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_select_write(FilterArgs a, const uint8_t *accept,
                                                      uint32_t n, const uint32_t *group_offset,
                                                      uint32_t *list)
{
    // stage[t]: sort key << 12 | the pair's offset in the group (< 4096)
    __shared__ uint32_t stage[SEL_PER_GROUP];
    __shared__ uint32_t hist[GK_MAX_READ_LEN + 1u];
    __shared__ uint32_t wave_sum[4], wave_min[4], wave_max[4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t i0 = blockIdx.x * SEL_PER_GROUP + threadIdx.x * SEL_PER_LANE;
    const uint32_t sel = select_bits<VEC>(accept, n, i0, nullptr, false);
    uint32_t k16[SEL_PER_LANE];
    length_keys(a, i0, sel, k16);
    const uint32_t c = (uint32_t)__popc(sel);
    uint32_t incl = c, lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        if (sel & (1u << j)) {
            lo = k16[j] < lo ? k16[j] : lo;
            hi = k16[j] > hi ? k16[j] : hi;
        }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o)
            incl += t;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t ol = __shfl_xor(lo, o, 64), oh = __shfl_xor(hi, o, 64);
        lo = ol < lo ? ol : lo;
        hi = oh > hi ? oh : hi;
    }
    if (lane == 63u)
        wave_sum[wave] = incl;
    if (lane == 0u) {
        wave_min[wave] = lo;
        wave_max[wave] = hi;
    }
    __syncthreads();
    const uint32_t total = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    uint32_t at = incl - c;
    for (uint32_t w = 0; w < wave; ++w)
        at += wave_sum[w];
    const uint32_t g0 = blockIdx.x * SEL_PER_GROUP;
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        if (sel & (1u << j))
            stage[at++] = (k16[j] << 12) | (i0 + j - g0);
    uint32_t kmin = wave_min[0], kmax = wave_max[0];
    for (uint32_t w = 1; w < 4u; ++w) {
        kmin = wave_min[w] < kmin ? wave_min[w] : kmin;
        kmax = wave_max[w] > kmax ? wave_max[w] : kmax;
    }
    const uint32_t nb = kmin < kmax ? kmax - kmin + 1u : 0u;
    for (uint32_t b = threadIdx.x; b < nb; b += 256u)
        hist[b] = 0u;
    __syncthreads();
    const uint32_t base = group_offset[blockIdx.x];
    if (nb == 0u) {                      // one key (or nothing listed): pair order
        for (uint32_t t = threadIdx.x; t < total; t += 256u)
            list[base + t] = g0 + (stage[t] & 4095u);
        return;
    }
    // Counting sort by key over [kmin, kmax] (the order within a key does not
    // matter: every result is written at its own pair index).
    for (uint32_t t = threadIdx.x; t < total; t += 256u)
        atomicAdd(&hist[(stage[t] >> 12) - kmin], 1u);
    __syncthreads();
    if (wave == 0u) {                    // exclusive prefix sums of the buckets
        const uint32_t per = (nb + 63u) / 64u;
        const uint32_t b0 = lane * per < nb ? lane * per : nb;
        const uint32_t b1 = b0 + per < nb ? b0 + per : nb;
        uint32_t sum = 0;
        for (uint32_t b = b0; b < b1; ++b)
            sum += hist[b];
        uint32_t run = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(run, o, 64);
            if (lane >= (uint32_t)o)
                run += t;
        }
        run -= sum;
        for (uint32_t b = b0; b < b1; ++b) {
            const uint32_t v = hist[b];
            hist[b] = run;
            run += v;
        }
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < total; t += 256u) {
        const uint32_t v = stage[t];
        list[base + atomicAdd(&hist[(v >> 12) - kmin], 1u)] = g0 + (v & 4095u);
    }
}

// ---- listing by (words of the read, e) over the whole batch ------------------
//
// With a threshold per pair a 4096-pair group lists a few hundred pairs over as
// many (words, e) bins, so sorting within groups leaves nearly every wave mixed.
// These kernels sort the listed pairs of the whole batch: each group counts its
// pairs per bin in LDS and adds the counts to one of BIN_COPIES copies of the
// bins' counts (by group number, so that no count is added to by more than
// 1 / BIN_COPIES of the groups); a scan turns the counts into starts, bin by bin
// and copy by copy; each group then reserves its run in its copy of each bin
// with one atomic and writes its pairs there (the order within a bin does not
// matter: every result is written at its own pair index).  Pairs that cannot be
// compared go to bin 0.
constexpr uint32_t BIN_COPIES = 32u;
constexpr uint32_t BIN_CELLS = VBINS * BIN_COPIES;   // counts, then cursors, then starts
static_assert(VERIFY_BIN_WORDS == 3u * BIN_CELLS, "the host allocates them");

__device__ __forceinline__ void bin_keys(const FilterArgs &a, uint32_t i0, uint32_t sel,
                                         uint32_t (&key)[SEL_PER_LANE])
{
    length_keys(a, i0, sel, key);
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j) {
        const uint32_t e = (sel & (1u << j)) ? (uint32_t)a.e_pair[i0 + j] : 0u;
        key[j] = key[j] && e <= GK_VERIFY_MAX_E ? ((key[j] + 31u) / 32u - 1u) * 32u + e : 0u;
    }
}

__global__ __launch_bounds__(256) void k_bin_zero(uint32_t *bins)
{
    for (uint32_t b = blockIdx.x * 256u + threadIdx.x; b < 2u * BIN_CELLS; b += gridDim.x * 256u)
        bins[b] = 0u;
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_bin_count(FilterArgs a, const uint8_t *accept, uint32_t n,
                                                   uint32_t *bins, uint16_t *dist)
{
    __shared__ uint32_t h[VBINS];
    for (uint32_t b = threadIdx.x; b < VBINS; b += 256u)
        h[b] = 0u;
    __syncthreads();
    const uint32_t i0 = blockIdx.x * SEL_PER_GROUP + threadIdx.x * SEL_PER_LANE;
    const uint32_t sel = select_bits<VEC>(accept, n, i0, dist, true);
    uint32_t key[SEL_PER_LANE];
    bin_keys(a, i0, sel, key);
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        if (sel & (1u << j))
            atomicAdd(&h[key[j]], 1u);
    __syncthreads();
    uint32_t *copy = bins + (blockIdx.x % BIN_COPIES) * VBINS;
    for (uint32_t b = threadIdx.x; b < VBINS; b += 256u)
        if (h[b])
            atomicAdd(&copy[b], h[b]);
}

// Starts of every (bin, copy) cell, bin-major, at bins[2 BIN_CELLS + copy *
// VBINS + bin], the total into *count.
__global__ __launch_bounds__(1024) void k_bin_scan(uint32_t *bins, uint32_t *count)
{
    __shared__ uint32_t wave_sum[16];
    constexpr uint32_t PER = BIN_CELLS / 1024u;       // cells per thread
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t local[PER], sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t cell = threadIdx.x * PER + q;  // = bin * BIN_COPIES + copy
        local[q] = bins[(cell % BIN_COPIES) * VBINS + cell / BIN_COPIES];
        sum += local[q];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o)
            incl += t;
    }
    if (lane == 63u)
        wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w)
        before += wave_sum[w];
    uint32_t run = before + incl - sum;
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t cell = threadIdx.x * PER + q;
        bins[2u * BIN_CELLS + (cell % BIN_COPIES) * VBINS + cell / BIN_COPIES] = run;
        run += local[q];
    }
    if (threadIdx.x == 1023u)
        *count = before + incl;
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_bin_write(FilterArgs a, const uint8_t *accept, uint32_t n,
                                                   uint32_t *bins, uint32_t *list)
{
    __shared__ uint32_t h[VBINS];
    for (uint32_t b = threadIdx.x; b < VBINS; b += 256u)
        h[b] = 0u;
    __syncthreads();
    const uint32_t i0 = blockIdx.x * SEL_PER_GROUP + threadIdx.x * SEL_PER_LANE;
    const uint32_t sel = select_bits<VEC>(accept, n, i0, nullptr, false);
    uint32_t key[SEL_PER_LANE], rank[SEL_PER_LANE];
    bin_keys(a, i0, sel, key);
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        rank[j] = (sel & (1u << j)) ? atomicAdd(&h[key[j]], 1u) : 0u;
    __syncthreads();
    // this group's run in its copy of each bin: the cell's start plus a
    // reservation on the cell's cursor
    const uint32_t c = (blockIdx.x % BIN_COPIES) * VBINS;
    for (uint32_t b = threadIdx.x; b < VBINS; b += 256u)
        if (h[b])
            h[b] = bins[2u * BIN_CELLS + c + b] + atomicAdd(&bins[BIN_CELLS + c + b], h[b]);
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < SEL_PER_LANE; ++j)
        if (sel & (1u << j))
            list[h[key[j]] + rank[j]] = i0 + j;
}

// Transposed read rows (word j of read r at reads[j * pitch + r]) to rows of
// `stride` words (a multiple of 4): a workgroup stages 256 reads in LDS (each
// row read with consecutive lanes on consecutive words), and each lane writes
// its read in 16-byte stores.  The list of a batch by (words, e) scatters each
// read's candidates, and a line per transposed row for each of them is what
// would bound their loads.
__global__ __launch_bounds__(256) void k_reads_rowwise(const uint32_t *reads, uint32_t pitch,
                                                       uint32_t rows, uint32_t n_reads,
                                                       uint32_t stride, uint32_t *out)
{
    extern __shared__ uint32_t lds_raw[];
    const uint32_t r = blockIdx.x * 256u + threadIdx.x;
    uint32_t *row = lds_raw + threadIdx.x * (stride + 1u);   // odd: distinct banks
    for (uint32_t j = 0; j < stride; ++j)
        row[j] = r < n_reads && j < rows ? reads[(size_t)j * pitch + r] : 0u;
    if (r < n_reads) {
        uint4 *q = reinterpret_cast<uint4 *>(out + (size_t)r * stride);
        for (uint32_t j = 0; j < stride; j += 4)
            q[j / 4] = make_uint4(row[j], row[j + 1], row[j + 2], row[j + 3]);
    }
}

// The list's pairs, 64 in a row per wave, by the tile form's algorithms on
// planes in LDS.  ROWWISE: the reads come from k_reads_rowwise.  Bound as the
// tile form by LDS latency (furthest-reaching points) and column steps (bands),
// but no wave is partly filled or mixes thresholds, and no LDS goes to the list:
// a workgroup more per compute unit at 8 to 10 words.  Figures at verify_lists.
template <int WMAX, int L, bool ROWWISE>
__global__ __launch_bounds__(256) void k_verify_waves(FilterArgs a, const uint32_t *list,
                                                      const uint32_t *count, uint16_t *dist,
                                                      uint32_t words)
{
    extern __shared__ uint32_t lds_raw[];
    const uint32_t lane = threadIdx.x & 63u;
    Column col;
    col.read = reinterpret_cast<uint2 *>(lds_raw) + (threadIdx.x >> 6) * wave_planes(words) + lane;
    col.text = col.read + (words + 1u) * 64u;
    const uint32_t n = *count;
    const uint32_t waves = gridDim.x * 4u;
    // the last bins, whose pairs take longest, first
    for (uint32_t c = blockIdx.x * 4u + (threadIdx.x >> 6); c * 64u < n; c += waves) {
        const uint32_t at = c * 64u + lane;
        const bool have = at < n;
        const uint32_t i = list[n - 1u - (have ? at : c * 64u)];
        const PairIdx p = load_idx(a, i);
        const bool live = have && p.r < a.n_reads && p.e <= GK_VERIFY_MAX_E;
        uint32_t len = a.read_len[live ? p.r : 0u];
        len = live && len <= a.max_read_len ? len : 0u;
        const uint32_t d = wave_distances<WMAX, L, ROWWISE>(a, p, len, col);
        if (have)
            dist[i] = (uint16_t)d;
    }
}

// Resident 256-lane workgroups per CU of k_verify_list.
template <int W, int L>
hipError_t list_blocks_per_cu(int &out)
{
    static int per_cu = -1;
    if (per_cu < 0) {
        int v = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &v, k_verify_list<W, L>, 256, 0);
        if (e != hipSuccess)
            return e;
        per_cu = v > 0 ? v : 1;
    }
    out = per_cu;
    return hipSuccess;
}

// The list of n pairs into x.list and its length into x.count; dist of the
// others set to GK_EST_NONE.
template <bool VEC>
void make_list(const FilterArgs &c, const uint8_t *accept, uint32_t n, uint16_t *dist,
               const VerifyScratch &x, hipStream_t s)
{
    const uint32_t groups = (n + SEL_PER_GROUP - 1) / SEL_PER_GROUP;
    if (c.e_pair) {
        hipLaunchKernelGGL(k_bin_zero, dim3(32), dim3(256), 0, s, x.bins);
        hipLaunchKernelGGL(k_bin_count<VEC>, dim3(groups), dim3(256), 0, s, c, accept, n, x.bins,
                           dist);
        hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, s, x.bins, x.count);
        hipLaunchKernelGGL(k_bin_write<VEC>, dim3(groups), dim3(256), 0, s, c, accept, n, x.bins,
                           x.list);
        return;
    }
    hipLaunchKernelGGL(k_select_count<VEC>, dim3(groups), dim3(256), 0, s, accept, n, x.groups,
                       dist);
    hipLaunchKernelGGL(k_select_scan, dim3(1), dim3(1024), 0, s, x.groups, groups, x.count);
    hipLaunchKernelGGL(k_select_write<VEC>, dim3(groups), dim3(256), 0, s, c, accept, n, x.groups,
                       x.list);
}

template <int W, int L>
hipError_t list_wl(const FilterArgs &c, uint16_t *dist, const VerifyScratch &x, uint32_t most,
                   int cus, hipStream_t s)
{
    int per_cu = 1;
    const hipError_t oe = list_blocks_per_cu<W, L>(per_cu);
    if (oe != hipSuccess)
        return oe;
    // Up to 8 times the resident workgroups: later workgroups start as
    // earlier ones finish, so the waves' gathers do not all come at once
    // (measured faster than one resident round at every sweep point; the
    // list length is only known on the device).
    const uint32_t grid = std::min(most, 8u * (uint32_t)(cus * per_cu));
    hipLaunchKernelGGL((k_verify_list<W, L>), dim3(grid), dim3(256), 0, s, c,
                       (const uint32_t *)x.list, (const uint32_t *)x.count, dist);
    return hipGetLastError();
}

template <int WMAX, int L, bool ROWWISE>
hipError_t waves_wl(const FilterArgs &c, uint16_t *dist, const VerifyScratch &x, uint32_t words,
                    uint32_t most, int cus, hipStream_t s)
{
    const uint32_t grid = std::min(most, 32u * (uint32_t)cus);
    hipLaunchKernelGGL((k_verify_waves<WMAX, L, ROWWISE>), dim3(grid), dim3(256),
                       4u * wave_planes(words) * sizeof(uint2), s, c, (const uint32_t *)x.list,
                       (const uint32_t *)x.count, dist, words);
    return hipGetLastError();
}

template <int L, bool ROWWISE>
hipError_t waves_l(const FilterArgs &c, uint16_t *dist, uint32_t words, const VerifyScratch &x,
                   uint32_t most, int cus, hipStream_t s)
{
    if (words <= 4)
        return waves_wl<4, L, ROWWISE>(c, dist, x, words, most, cus, s);
    if (words <= 8)
        return waves_wl<8, L, ROWWISE>(c, dist, x, words, most, cus, s);
    if (words <= 10)
        return waves_wl<10, L, ROWWISE>(c, dist, x, words, most, cus, s);
    return waves_wl<16, L, ROWWISE>(c, dist, x, words, most, cus, s);
}

// Distances of the list's pairs.
template <int L>
hipError_t list_l(const FilterArgs &c, uint16_t *dist, uint32_t words, const VerifyScratch &x,
                  uint32_t most, int cus, hipStream_t s)
{
    if (c.e_pair) {
        FilterArgs r = c;
        r.reads = x.reads;
        r.pitch = verify_read_stride(c.rows);
        return waves_l<L, true>(r, dist, words, x, most, cus, s);
    }
    if (c.e_uniform <= FURTHEST_MAX_E)
        return waves_l<L, false>(c, dist, words, x, most, cus, s);
    switch (words) {
    case 1: return list_wl<1, L>(c, dist, x, most, cus, s);
    case 2: return list_wl<2, L>(c, dist, x, most, cus, s);
    case 3: return list_wl<3, L>(c, dist, x, most, cus, s);
    case 4: return list_wl<4, L>(c, dist, x, most, cus, s);
    case 5: return list_wl<5, L>(c, dist, x, most, cus, s);
    case 6: return list_wl<6, L>(c, dist, x, most, cus, s);
    case 7: return list_wl<7, L>(c, dist, x, most, cus, s);
    case 8: return list_wl<8, L>(c, dist, x, most, cus, s);
    case 9: return list_wl<9, L>(c, dist, x, most, cus, s);
    case 10: return list_wl<10, L>(c, dist, x, most, cus, s);
    case 11: return list_wl<11, L>(c, dist, x, most, cus, s);
    case 12: return list_wl<12, L>(c, dist, x, most, cus, s);
    case 13: return list_wl<13, L>(c, dist, x, most, cus, s);
    case 14: return list_wl<14, L>(c, dist, x, most, cus, s);
    case 15: return list_wl<15, L>(c, dist, x, most, cus, s);
    case 16: return list_wl<16, L>(c, dist, x, most, cus, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_verify(const FilterArgs &a, const uint8_t *accept, uint16_t *dist,
                         uint32_t words, uint32_t layout, hipStream_t s)
{
    const uint32_t tile = tile_of(a.n_pairs, words);
    return layout == GK_READS_INTERLEAVED
               ? tile_l<GK_READS_INTERLEAVED>(a, accept, dist, words, tile, s)
               : tile_l<GK_READS_SPLIT>(a, accept, dist, words, tile, s);
}

hipError_t launch_verify_listed(const FilterArgs &a, const uint8_t *accept, uint16_t *dist,
                                uint32_t words, uint32_t layout, const VerifyScratch &x, int cus,
                                hipStream_t s)
{
    if (a.e_pair) {
        const uint32_t stride = verify_read_stride(a.rows);
        hipLaunchKernelGGL(k_reads_rowwise, dim3((a.n_reads + 255u) / 256u), dim3(256),
                           256u * (stride + 1u) * sizeof(uint32_t), s, a.reads, a.pitch, a.rows,
                           a.n_reads, stride, x.reads);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    const uint64_t CHUNK = 1ull << 30;
    for (uint64_t first = 0; first < a.n_pairs; first += CHUNK) {
        FilterArgs c = a;
        const uint64_t n = a.n_pairs - first < CHUNK ? a.n_pairs - first : CHUNK;
        c.n_pairs = n;
        c.pair_read = a.pair_read ? a.pair_read + first : nullptr;
        if (!a.pair_read && first > 0)
            c.n_reads = 0;   // pair i uses read i < n_reads < 2^30: none here
        c.cand_pos = a.cand_pos + first;
        c.e_pair = a.e_pair ? a.e_pair + first : nullptr;
        c.accept = nullptr;
        c.est = nullptr;
        c.accept_bits = nullptr;
        const uint8_t *acc = accept ? accept + first : nullptr;
        uint16_t *out = dist + first;
        if (((uintptr_t)acc & 15u) == 0 && ((uintptr_t)out & 15u) == 0)
            make_list<true>(c, acc, (uint32_t)n, out, x, s);
        else
            make_list<false>(c, acc, (uint32_t)n, out, x, s);
        hipError_t e = hipGetLastError();
        const uint32_t most = (uint32_t)((n + 255) / 256);
        if (e == hipSuccess)
            e = layout == GK_READS_INTERLEAVED
                    ? list_l<GK_READS_INTERLEAVED>(c, out, words, x, most, cus, s)
                    : list_l<GK_READS_SPLIT>(c, out, words, x, most, cus, s);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace gkd
