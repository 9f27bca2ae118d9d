// Mixed-batch GateKeeper-GPU filter for gfx950: one launch over a batch whose
// pairs differ in read length and threshold.
//
// The paper fixes the read length and e at compile time (Sec. 3.1, 3.2) and
// so runs one kernel per (length, e) group.  Here workgroups take the batch in
// tiles of T consecutive pairs:
//   - a workgroup classifies the tile's pairs (invalid and undefined pairs are
//     done at once, pairs with more than 31 shifts are set apart) and
//     counting-sorts the rest in LDS by (words per mask W, k_max), so that a
//     64-lane chunk holds one W and nearly equal e;
//   - its waves take chunks from an LDS counter and run the register-only
//     fast path of gk_pair.h for the chunk's W (a wave-uniform switch), one
//     or two pairs per lane (two: both pairs' loads in flight before either
//     is computed; only for up to 10 words per mask, where the registers for
//     it fit); a pair's entry (read, position, length, e) stays in LDS from
//     the classification on, and its result takes the entry's place until the
//     tile is written back in slot order (results land in sorted order, so
//     writing them directly would scatter partial-line writes).
// Pairs with more than 31 shifts are a tile's last chunks, on the general path.
// Two forms:
//   direct      one batch, one workgroup per tile, accept bits with the
//               results: one launch, no scratch;
//   table       resident workgroups claim tiles of a table of batches from a
//               device counter, so that one captured graph serves any batches;
//   inline      one workgroup per tile of a table that comes with the kernel's
//               arguments;
//   ordered     the direct form for the plain call, which cannot know whether
//               the thresholds of an array differ: a tile whose pairs lie in
//               runs of one (W, k_max) goes to the chunks unsorted (a constant
//               threshold over 2^20 pairs of 150 bases, e = 3: 25 us, 32 sorted,
//               24 without looking; 2^22 of 250, e = 1: 87, 106 and 102), and
//               widths of 6, 8 and 12 words keep the waves per SIMD of the plain
//               kernel (5, 4 and 3, against 4, 4 and 2 in the next wider) and
//               the general path, where all pairs take it, near the read's width
//               (2^20 pairs of 200 bases, e = 32 to 59: 358 us, 435 at 10 words).
#include "gk_pair.h"

namespace gkd {

namespace {

constexpr uint32_t NBINS = 16 * 32;       // W in 1..16, k_max in 0..31
constexpr uint32_t FAR = 16;              // chunk class of the pairs with more shifts

struct MixedLds {
    uint32_t hist[NBINS + 1];             // bin NBINS: class FAR
    uint32_t wstart[18];
    uint32_t tile;
    uint32_t n_chunks;
    uint32_t next_chunk;
    uint32_t sorts;                       // 0: every 64 pairs in a row share a bin
    uint32_t pad_;
};

// Dynamic LDS after MixedLds: the tile's pair entries pos[T], read[T],
// entry[T] u32, chunk_start[C] u32, chunk_info[C] u32 with C = T/64 + 17
// (T/64 times the lanes per pair), sorted[T] u16 (first the pairs' sort keys,
// then the slots in sorted order).
__host__ __device__ inline uint32_t mixed_chunk_cap(uint32_t tile, uint32_t lg)
{
    return (tile << lg) / 64 + 17;
}

__host__ inline size_t mixed_lds_bytes(uint32_t tile, uint32_t lg = 0)
{
    return sizeof(MixedLds) + 12u * tile + 8u * mixed_chunk_cap(tile, lg) + 2u * tile;
}

// The tile's pairs: entry[slot] is e | length << 8 until the pair is done, then
// its result code | estimate << 16.
struct TilePairs {
    uint32_t *pos, *read, *entry;
};

__device__ __forceinline__ void tile_done(const TilePairs &t, uint32_t slot, uint32_t res,
                                          uint32_t est)
{
    t.entry[slot] = res | (est << 16);
}

// Loads of a classified pair (its length is known, its read holds no unknown
// base).
template <int W>
__device__ __forceinline__ PairIdx load_slot(const FilterArgs &a, const TilePairs &t,
                                             uint32_t slot, PairData<W> &d)
{
    PairIdx p;
    const uint32_t en = t.entry[slot];
    p.r = t.read[slot];
    p.pos = t.pos[slot];
    p.e = en & 0xFFu;
    load_words<W>(a, p.r, d);
    load_window<W>(a, p.pos, d);
    load_unknown_lines<W>(a, p.pos, d);
    d.m = en >> 8;
    d.has_n = 0u;
    return p;
}

template <int W, int L, bool GENERAL, bool VAR, bool SPLIT>
__device__ __forceinline__ void run_chunk_pair(const FilterArgs &a, const TilePairs &t,
                                               uint32_t slot, uint32_t sub, uint32_t lanes)
{
    PairData<W> d;
    const PairIdx p = load_slot<W>(a, t, slot, d);
    uint32_t est;
    const uint32_t res = compute_pair<W, L, GENERAL, VAR, false, SPLIT>(a, p, d, est, sub, lanes);
    if (sub == 0u)
        tile_done(t, slot, res, est);
}

template <int W, int L, bool VAR>
__device__ __forceinline__ void run_chunk_pair2(const FilterArgs &a, const TilePairs &t,
                                                uint32_t s0, bool has1, uint32_t s1)
{
    // both pairs' loads in flight before either is computed
    PairData<W> d0, d1;
    const PairIdx p0 = load_slot<W>(a, t, s0, d0);
    const PairIdx p1 = load_slot<W>(a, t, has1 ? s1 : s0, d1);
    uint32_t est;
    uint32_t res = compute_pair<W, L, false, VAR>(a, p0, d0, est);
    tile_done(t, s0, res, est);
    if (has1) {
        res = compute_pair<W, L, false, VAR>(a, p1, d1, est);
        tile_done(t, s1, res, est);
    }
}

template <int WMAX, int L, int PPL, bool VAR, bool SPLIT>
__device__ __forceinline__ void run_chunk(const FilterArgs &a, const TilePairs &t, uint32_t w,
                                          uint32_t s0, bool has1, uint32_t s1, uint32_t sub,
                                          uint32_t lanes)
{
#define GK_CASE(N)                                                                 \
    case N:                                                                        \
        if (N <= WMAX) {                                                           \
            if (PPL == 2)                                                          \
                run_chunk_pair2<(N <= WMAX ? N : 1), L, VAR>(a, t, s0, has1, s1);  \
            else                                                                   \
                run_chunk_pair<(N <= WMAX ? N : 1), L, false, VAR, SPLIT>(a, t, s0, sub, lanes); \
        }                                                                          \
        break;
    switch (w) {
        GK_CASE(1) GK_CASE(2) GK_CASE(3) GK_CASE(4) GK_CASE(5) GK_CASE(6) GK_CASE(7) GK_CASE(8)
        GK_CASE(9) GK_CASE(10) GK_CASE(11) GK_CASE(12) GK_CASE(13) GK_CASE(14) GK_CASE(15)
        GK_CASE(16)
    default:
        break;
    }
#undef GK_CASE
}

enum Form { DIRECT, TABLE, INLINE, ORDERED };

// Batch of a tile in a table launch: the last b with prefix[b] <= tile (empty
// batches share their prefix with the next one, so the last match is the
// batch that owns the tile).
template <typename Table>
__device__ __forceinline__ uint32_t table_batch(const Table *t, uint32_t tile)
{
    uint32_t lo = 0, hi = t->n_batches;          // prefix[hi] > tile
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (t->prefix[mid] <= tile)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Arguments of batch b (uniform), by scalar loads: nothing writes the table
// while a launch reads it.
__device__ __forceinline__ FilterArgs table_args(const BatchTable *t, uint32_t b)
{
    typedef const __attribute__((address_space(4))) uint32_t *constant_words;
    static_assert(sizeof(FilterArgs) % 4 == 0, "copied as words");
    const constant_words src = (constant_words)(uintptr_t)&t->args[b];
    uint32_t w[sizeof(FilterArgs) / 4];
#pragma unroll
    for (uint32_t k = 0; k < sizeof(FilterArgs) / 4; ++k)
        w[k] = src[k];
    FilterArgs a;
    __builtin_memcpy(&a, w, sizeof a);
    return a;
}

// SPLIT: a small batch, 2^x.lg lanes per pair (split_lanes).
struct NoTable {};

template <int WMAX, int L, int PPL, bool VAR = false, Form FORM = TABLE, bool SPLIT = false,
          typename Batches = NoTable>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(WMAX <= 10 && PPL == 1 && !VAR && !SPLIT ? 4 : 1)))
void k_mixed(FilterArgs a0, MixedArgs x, Batches batches)
{
    extern __shared__ uint32_t lds_raw[];
    MixedLds &s = *reinterpret_cast<MixedLds *>(lds_raw);
    TilePairs t;
    t.pos = lds_raw + sizeof(MixedLds) / 4;
    t.read = t.pos + x.tile;
    t.entry = t.read + x.tile;
    uint32_t *chunk_start = t.entry + x.tile;
    uint32_t *chunk_info = chunk_start + mixed_chunk_cap(x.tile, SPLIT ? x.lg : 0u);
    uint16_t *sorted = reinterpret_cast<uint16_t *>(chunk_info + mixed_chunk_cap(x.tile, SPLIT ? x.lg : 0u));

    while (true) {
        // (not known to be the same in the next tile's round, so that nothing
        // derived from it is held in registers across the chunks)
        uint32_t tid = threadIdx.x;
        if (FORM == TABLE)
            asm volatile("" : "+v"(tid));
        const uint32_t lane = tid & 63u;
        if (FORM == TABLE && tid == 0)
            s.tile = atomicAdd(x.tile_counter, 1u);
        for (uint32_t b = tid; b <= NBINS; b += 256)
            s.hist[b] = 0;
        if (FORM == ORDERED && tid == 0)
            s.sorts = 0u;
        __syncthreads();
        FilterArgs a = a0;
        uint32_t base = blockIdx.x * x.tile, batch = 0;
        if constexpr (FORM == INLINE) {
            batch = __builtin_amdgcn_readfirstlane(table_batch(&batches, blockIdx.x));
            a = batches.args[batch];
            base = (blockIdx.x - batches.prefix[batch]) * x.tile;
        }
        if constexpr (FORM == TABLE) {
            // uniform, so that the batch's arguments come into scalar registers
            const uint32_t tile = __builtin_amdgcn_readfirstlane(s.tile);
            if (tile >= x.table->prefix[x.table->n_batches])
                break;
            batch = __builtin_amdgcn_readfirstlane(table_batch(x.table, tile));
            a = table_args(x.table, batch);
            base = (tile - x.table->prefix[batch]) * x.tile;
        }
        const uint32_t n = (uint32_t)a.n_pairs;

        // 1. classify, four pairs' loads in flight per lane
        for (uint32_t j0 = tid; j0 < x.tile; j0 += 1024) {
            PairIdx p[4];
            uint32_t m[4], un[4];
            // (a tile of 512 has two: no loads for the others)
            const bool four = FORM != ORDERED || x.tile > 512u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < 2 || four) {
                    const uint32_t i = base + j0 + 256u * q;
                    p[q] = load_idx(a, i < n ? i : n - 1u);
                }
            }
            const uint8_t *flag = a.read_has_n ? a.read_has_n
                                               : reinterpret_cast<const uint8_t *>(a.read_len);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < 2 || four) {
                    const uint32_t r = p[q].r < a.n_reads ? p[q].r : 0u;
                    m[q] = a.read_len[r];
                    un[q] = flag[r];
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t j = j0 + 256u * q;
                if (j >= x.tile)
                    break;
                m[q] = p[q].r < a.n_reads ? m[q] : 0u;
                uint32_t en = GK_INVALID | (GK_EST_NONE << 16), key = NBINS + 1;
                if (base + j >= n || m[q] == 0u || m[q] > a.max_read_len) {
                } else if ((uint64_t)p[q].pos + m[q] > a.ref_len || (a.read_has_n && un[q])) {
                    en = GK_UNDEFINED | (GK_EST_NONE << 16);
                } else {
                    const uint32_t kmax = p[q].e < m[q] - 1u ? p[q].e : m[q] - 1u;
                    const uint32_t w = (m[q] + 31u) / 32u;
                    en = p[q].e | (m[q] << 8);
                    key = kmax <= 31u ? (w - 1u) * 32u + (x.sort_e ? kmax : 0u) : NBINS;
                }
                t.pos[j] = p[q].pos;
                t.read[j] = p[q].r;
                t.entry[j] = en;
                sorted[j] = (uint16_t)key;         // until step 3
                if constexpr (FORM != ORDERED) {
                    if (key <= NBINS)
                        atomicAdd(&s.hist[key], 1u);
                    continue;
                }
                // one bin for the wave's 64 pairs: counted at once
                const unsigned long long on = __ballot(key <= NBINS);
                if (on == 0ull)
                    continue;
                const uint32_t first = __builtin_ctzll(on);
                const uint32_t key0 = __builtin_amdgcn_readlane(key, first);
                if (__ballot(key <= NBINS && key != key0) == 0ull) {
                    if (lane == first)
                        atomicAdd(&s.hist[key], (uint32_t)__builtin_popcountll(on));
                } else {
                    if (key <= NBINS)
                        atomicAdd(&s.hist[key], 1u);
                    s.sorts = 1u;
                }
            }
        }
        __syncthreads();
        const bool sorts = FORM != ORDERED || __builtin_amdgcn_readfirstlane(s.sorts) != 0u;

        if (sorts) {
            // 2. exclusive prefix over the bins (wave 0: 8 bins per lane)
            if (tid < 64) {
                uint32_t local[8], sum = 0;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    local[q] = s.hist[tid * 8 + q];
                    sum += local[q];
                }
                uint32_t incl = sum;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t v = __shfl_up(incl, o, 64);
                    if (lane >= (uint32_t)o)
                        incl += v;
                }
                uint32_t run = incl - sum;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint32_t b = tid * 8 + q;
                    if (b % 32u == 0u)
                        s.wstart[b / 32u] = run;
                    s.hist[b] = run;
                    run += local[q];
                }
                if (tid == 63) {
                    s.wstart[FAR] = run;
                    s.wstart[FAR + 1] = run + s.hist[NBINS];
                    s.hist[NBINS] = run;
                }
            }
            // keys to registers: the sorted slots take their place
            uint32_t key8[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t j = tid + 256u * q;
                key8[q] = j < x.tile ? sorted[j] : NBINS + 1u;
            }
            __syncthreads();

            // 3. scatter slots into bin order
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (key8[q] <= NBINS)
                    sorted[atomicAdd(&s.hist[key8[q]], 1u)] = (uint16_t)(tid + 256u * q);

            // 4. chunks: runs of one W, 64 * ppl pairs at most.  A W's pairs are
            //    in ascending k_max, so its one partial chunk is put first, on the
            //    pairs with the fewest shifts: its idle lanes then wait through
            //    the shortest loop.
            if (tid < 64) {
                const uint32_t ch = SPLIT ? 64u >> x.lg : tid == FAR ? 64u : 64u * PPL;
                const uint32_t w0 = tid <= FAR ? s.wstart[tid] : 0u;
                const uint32_t cnt = tid <= FAR ? s.wstart[tid + 1] - w0 : 0u;
                const uint32_t nch = (cnt + ch - 1) / ch;
                const uint32_t lead = cnt % ch == 0u ? ch : cnt % ch;   // size of chunk 0
                uint32_t incl = nch;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t v = __shfl_up(incl, o, 64);
                    if (lane >= (uint32_t)o)
                        incl += v;
                }
                const uint32_t first = incl - nch;
                for (uint32_t c = 0; c < nch; ++c) {
                    chunk_start[first + c] = w0 + (c == 0u ? 0u : lead + (c - 1u) * ch);
                    chunk_info[first + c] = (c == 0u ? lead : ch) | ((tid + 1u) << 16);
                }
                if (tid == 63) {
                    s.n_chunks = incl;
                    s.next_chunk = 0;
                }
            }
            __syncthreads();
        }

        // 5. waves take chunks, the heaviest (largest W and k_max, at the
        //    end of the list) first, so the tile ends on short chunks; of a
        //    tile left in order each its own 64 pairs
        const uint32_t lanes = SPLIT ? 1u << x.lg : 1u, sub = lane & (lanes - 1u);
        const uint32_t n_chunks = sorts ? s.n_chunks : x.tile * lanes / 64u;
        uint32_t own = __builtin_amdgcn_readfirstlane(tid >> 6);
        while (true) {
            uint32_t c = own;
            if (sorts) {
                if (lane == 0)
                    c = atomicAdd(&s.next_chunk, 1u);
                c = __builtin_amdgcn_readfirstlane(c);
            }
            own += 4u;
            if (c >= n_chunks)
                break;
            uint32_t at = SPLIT ? lane >> x.lg : lane, cnt, w, s0;
            bool on;
            if (sorts) {
                c = n_chunks - 1u - c;
                const uint32_t start = __builtin_amdgcn_readfirstlane(chunk_start[c]);
                const uint32_t info = __builtin_amdgcn_readfirstlane(chunk_info[c]);
                cnt = info & 0xFFFFu;
                w = info >> 16;
                on = at < cnt;
                at += start;
                s0 = on ? sorted[at] : 0u;
            } else {
                cnt = 0u;
                s0 = at + c * 64u / lanes;
                const uint32_t key = sorted[s0];
                on = key <= NBINS;
                const unsigned long long any = __ballot(on);
                if (any == 0ull)
                    continue;
                const uint32_t key0 = __builtin_amdgcn_readlane(key, __builtin_ctzll(any));
                w = key0 == NBINS ? FAR + 1u : key0 / 32u + 1u;
            }
            // The arguments anew for each chunk: what all 16 widths derive from
            // them (row addresses above all) does not fit the scalar registers
            // when the compiler computes it before the loop.
            FilterArgs a = a0;
            if constexpr (FORM != DIRECT)
                asm volatile("" : "+s"(batch));
            if constexpr (FORM == TABLE)
                a = table_args(x.table, batch);
            if constexpr (FORM == INLINE)
                a = batches.args[batch];
            asm volatile("" : "+s"(a.pitch), "+s"(a.rows), "+s"(a.max_read_len));
            if (on) {
                if (w == FAR + 1u) {
                    run_chunk_pair<WMAX, L, true, VAR, SPLIT>(a, t, s0, sub, lanes);
                } else {
                    const bool has1 = PPL == 2 && lane + 64u < cnt;
                    const uint32_t s1 = has1 ? sorted[at + 64u] : s0;
                    run_chunk<WMAX, L, PPL, VAR, SPLIT>(a, t, w, s0, has1, s1, sub, lanes);
                }
            }
        }
        __syncthreads();

        // 6. write the tile's results back in slot order
        const uint32_t live = n - base < x.tile ? n - base : x.tile;
        for (uint32_t j = tid; j < x.tile; j += 256) {
            const uint32_t v = t.entry[j];
            if (j < live) {
                a.accept[base + j] = (uint8_t)v;
                a.est[base + j] = (uint16_t)(v >> 16);
            }
            if (a.accept_bits) {
                const uint32_t res = v & 0xFFu;
                const unsigned long long bits =
                    __ballot(j < live && (res == GK_ACCEPT || res == GK_UNDEFINED));
                if (lane == 0u && j < live)
                    a.accept_bits[(base + j) >> 6] = bits;
            }
        }
        if (FORM != TABLE)
            break;
        __syncthreads();
    }
}

__global__ __launch_bounds__(64) void k_reset(uint32_t *tile_counter)
{
    if (threadIdx.x == 0)
        *tile_counter = 0;
}

// ORD: the ordered form.
template <int WMAX, int L, bool ORD = false>
hipError_t launch_mixed_wl(const FilterArgs &a, const MixedArgs &x, hipStream_t s)
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
        c.accept = a.accept + first;
        c.est = a.est + first;
        c.accept_bits = a.accept_bits ? a.accept_bits + first / 64 : nullptr;
        const dim3 grid((uint32_t)((n + x.tile - 1) / x.tile));
        const size_t lds = mixed_lds_bytes(x.tile, x.lg);
        auto kernel = k_mixed<WMAX, L, 1, false, ORD ? ORDERED : DIRECT>;
        if constexpr (!ORD) {
            if (a.flags != 0u)            // variant semantics: their own kernel
                kernel = k_mixed<WMAX, L, 1, true, DIRECT>;
            else if (x.lg != 0u)
                kernel = k_mixed<WMAX, L, 1, false, DIRECT, true>;
            if constexpr (WMAX <= 10)
                if (x.ppl == 2 && x.lg == 0u && a.flags == 0u)
                    kernel = k_mixed<WMAX, L, 2, false, DIRECT>;
        }
        hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, c, x, NoTable{});
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <int WMAX, int L>
hipError_t launch_table_wl(const MixedArgs &x, hipStream_t s)
{
    FilterArgs none{};
    if (x.n_tiles != 0u) {
        const BatchTable *t = x.table;
        InlineTable in;
        if (t->n_batches > INLINE_BATCHES || t->prefix[t->n_batches] != x.n_tiles)
            return hipErrorInvalidValue;
        in.n_batches = t->n_batches;
        for (uint32_t b = 0; b < t->n_batches; ++b) {
            in.prefix[b] = t->prefix[b];
            in.args[b] = t->args[b];
        }
        in.prefix[t->n_batches] = x.n_tiles;
        hipLaunchKernelGGL((k_mixed<WMAX, L, 1, false, INLINE, false, InlineTable>),
                           dim3(x.n_tiles), dim3(256), mixed_lds_bytes(x.tile), s, none, x, in);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, s, x.tile_counter);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if constexpr (WMAX <= 10) {
        if (x.ppl == 2) {
            hipLaunchKernelGGL((k_mixed<WMAX, L, 2>), dim3(x.blocks), dim3(256),
                               mixed_lds_bytes(x.tile), s, none, x, NoTable{});
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_mixed<WMAX, L, 1>), dim3(x.blocks), dim3(256), mixed_lds_bytes(x.tile),
                       s, none, x, NoTable{});
    return hipGetLastError();
}

template <int L>
hipError_t launch_mixed_l(const FilterArgs &a, const MixedArgs &x, uint32_t wmax, hipStream_t s)
{
    if (wmax <= 4)
        return launch_mixed_wl<4, L>(a, x, s);
    if (wmax <= 10)
        return launch_mixed_wl<10, L>(a, x, s);
    return launch_mixed_wl<16, L>(a, x, s);
}

template <int L>
hipError_t launch_ordered_l(const FilterArgs &a, const MixedArgs &x, uint32_t wmax, hipStream_t s)
{
    if (wmax <= 6)
        return launch_mixed_wl<6, L, true>(a, x, s);
    if (wmax <= 8)
        return launch_mixed_wl<8, L, true>(a, x, s);
    if (wmax <= 10)
        return launch_mixed_wl<10, L, true>(a, x, s);
    if (wmax <= 12)
        return launch_mixed_wl<12, L, true>(a, x, s);
    return launch_mixed_wl<16, L, true>(a, x, s);
}

template <int WMAX, int L>
hipError_t occupancy_wl(uint32_t tile, uint32_t ppl, int *blocks_per_cu)
{
    if constexpr (WMAX <= 10) {
        if (ppl == 2)
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                blocks_per_cu, k_mixed<WMAX, L, 2>, 256, mixed_lds_bytes(tile));
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_mixed<WMAX, L, 1>, 256,
                                                        mixed_lds_bytes(tile));
}

}  // namespace

hipError_t mixed_blocks_per_cu(uint32_t wmax, uint32_t layout, uint32_t tile, uint32_t ppl,
                               int *out)
{
    const bool il = layout == GK_READS_INTERLEAVED;
    if (wmax <= 4)
        return il ? occupancy_wl<4, GK_READS_INTERLEAVED>(tile, ppl, out)
                  : occupancy_wl<4, GK_READS_SPLIT>(tile, ppl, out);
    if (wmax <= 10)
        return il ? occupancy_wl<10, GK_READS_INTERLEAVED>(tile, ppl, out)
                  : occupancy_wl<10, GK_READS_SPLIT>(tile, ppl, out);
    return il ? occupancy_wl<16, GK_READS_INTERLEAVED>(tile, ppl, out)
              : occupancy_wl<16, GK_READS_SPLIT>(tile, ppl, out);
}

hipError_t launch_mixed_table(const MixedArgs &x, uint32_t wmax, uint32_t layout, hipStream_t s)
{
    const bool il = layout == GK_READS_INTERLEAVED;
    if (wmax <= 4)
        return il ? launch_table_wl<4, GK_READS_INTERLEAVED>(x, s)
                  : launch_table_wl<4, GK_READS_SPLIT>(x, s);
    if (wmax <= 10)
        return il ? launch_table_wl<10, GK_READS_INTERLEAVED>(x, s)
                  : launch_table_wl<10, GK_READS_SPLIT>(x, s);
    return il ? launch_table_wl<16, GK_READS_INTERLEAVED>(x, s)
              : launch_table_wl<16, GK_READS_SPLIT>(x, s);
}

hipError_t launch_mixed(const FilterArgs &a, const MixedArgs &x, uint32_t wmax, uint32_t layout,
                        hipStream_t s)
{
    return layout == GK_READS_INTERLEAVED
               ? launch_mixed_l<GK_READS_INTERLEAVED>(a, x, wmax, s)
               : launch_mixed_l<GK_READS_SPLIT>(a, x, wmax, s);
}

hipError_t launch_ordered(const FilterArgs &a, uint32_t wmax, uint32_t layout, hipStream_t s)
{
    MixedArgs x{};
    x.tile = filter_tile(a.n_pairs);
    x.ppl = 1;
    x.sort_e = 1;
    return layout == GK_READS_INTERLEAVED
               ? launch_ordered_l<GK_READS_INTERLEAVED>(a, x, wmax, s)
               : launch_ordered_l<GK_READS_SPLIT>(a, x, wmax, s);
}

}  // namespace gkd
