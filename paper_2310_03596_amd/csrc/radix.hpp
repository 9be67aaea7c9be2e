// Stable least-significant-digit radix sort of (key, index) pairs held in the
// workspace, with digits of 8 to 10 bits chosen so that a key takes as few
// passes as possible (two for keys of up to 20 bits).  Each pass: (1)
// per-tile digit histograms in LDS, (2) one workgroup per digit scans that
// digit's counts over tiles (not in small sorts), (3) each tile ranks its keys stably with
// wavefront ballots (one ballot per digit bit gives every lane the mask of
// lanes holding the same digit; popcount of the lanes below gives the rank
// inside the wavefront) and scatters.  Used for the bucket sort (Section I)
// and the sort by balancing hash (Section III.A).
#pragma once
#include "common.hpp"

namespace sph {

namespace {

#ifndef SPH_SORT_WIDE
#define SPH_SORT_WIDE 2
#endif
// Keys per thread of a tile: 10-bit digits take tiles SPH_SORT_WIDE times as
// long, so the per-tile work that scales with the 1024 digits (clearing and
// writing the tile's histogram, reading it back for the scatter) stays small
// next to the keys (measured on 8 M + 2 M keys: 2 and 4 equal, both 5 %
// faster than 1).
template <int D>
constexpr int sort_items = D >= 10 ? SPH_SORT_WIDE * kSortItems : kSortItems;

__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        uint32_t t = __shfl_up(v, off, kWave);
        if (lane >= off) v += t;
    }
    return v;
}

// Orders this wavefront's LDS accesses before its following ones.
__device__ inline void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive scan over the NT threads of a block; every thread gets `total`.
template <int NT = kBlock>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t &total)
{
    __shared__ uint32_t wsum[NT / kWave];
    int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t inc = wave_incl_scan(v);
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        uint32_t s = wsum[w];
        before += (w < wave) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return before + inc - v;
}

// In-place exclusive scan of row[0, len) by one block of NT threads; returns
// the row's total.  The row is taken in tiles of NT * B entries: a tile is
// loaded with coalesced reads (all in flight at once) into LDS, each thread
// then scans B consecutive entries of it (entry e sits at e + e / B, so the
// threads' strided LDS reads hit distinct banks), one block scan gives every
// thread its offset, and the tile is written back coalesced.  A tile costs
// one memory round trip and one block scan, where a scan 256 entries at a
// time costs one of each per 256 entries.
template <int NT, int B>
__device__ inline uint32_t block_scan_row(uint32_t *__restrict__ row, uint32_t len)
{
    constexpr uint32_t T = (uint32_t)NT * B;
    __shared__ uint32_t sh[T + T / B];
    const uint32_t tid = threadIdx.x;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < len; base += T) {
        uint32_t q[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const uint32_t e = (uint32_t)k * NT + tid;
            q[k] = base + e < len ? row[base + e] : 0u;
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const uint32_t e = (uint32_t)k * NT + tid;
            sh[e + e / B] = q[k];
        }
        __syncthreads();
        uint32_t v[B];
        uint32_t sum = 0;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            v[u] = sh[tid * (B + 1) + u];
            sum += v[u];
        }
        uint32_t tot;
        uint32_t run = carry + block_excl_scan<NT>(sum, tot);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            sh[tid * (B + 1) + u] = run;
            run += v[u];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const uint32_t e = (uint32_t)k * NT + tid;
            if (base + e < len) row[base + e] = sh[e + e / B];
        }
        carry += tot;
        __syncthreads();   // the next tile overwrites the LDS copy
    }
    return carry;
}

// Adds one chunk of a tile (the kBlock keys' digits d, BINS for no key) to
// the tile's histogram h in LDS.  Runs of equal digits in consecutive lanes
// add their length once (the keys arrive nearly sorted, step after step, so
// runs are long and the LDS atomics do not serialise on one address).
template <int D>
__device__ inline void hist_chunk(uint32_t *h, uint32_t d, bool valid)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t prev = __shfl_up(d, 1, kWave);
    const bool head = lane == 0 || d != prev;
    const uint64_t heads = __ballot(head);
    const uint64_t above = heads & ~((2ull << lane) - 1ull);   // heads past this lane (2 << 63 wraps to 0)
    const int next = above ? __ffsll((unsigned long long)above) - 1 : kWave;
    if (valid && head) atomicAdd(&h[d], (uint32_t)(next - lane));
}

// A tile's digit counts lie in one run per tile where the scatter adds up the
// tiles' counts itself (few tiles), and digit by digit where a kernel scans
// each digit's counts over the tiles first.
template <int D>
__device__ inline size_t hist_at(uint32_t digit, uint32_t tile, uint32_t tiles, bool by_tile)
{
    return by_tile ? (size_t)tile * (1u << D) + digit : (size_t)digit * tiles + tile;
}

template <int D, int IT>
__global__ __launch_bounds__(kBlock) void k_upsweep(const uint32_t *__restrict__ keys, uint32_t n, int shift,
                                                    uint32_t *__restrict__ hist, uint32_t tiles, bool by_tile)
{
    constexpr int BINS = 1 << D;
    __shared__ uint32_t h[BINS];
    for (int b = threadIdx.x; b < BINS; b += kBlock) h[b] = 0;
    __syncthreads();
    // Consecutive tiles run on one XCD: a digit's counts of 32 consecutive
    // tiles share one 128-byte line of hist, which is then written (here)
    // and read (in the scatter) through a single L2 instead of eight.
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t base = tile * (kBlock * IT);
    uint32_t keyv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const uint32_t e = base + it * kBlock + threadIdx.x;
        keyv[it] = e < n ? keys[e] : 0u;
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const uint32_t e = base + it * kBlock + threadIdx.x;
        const bool valid = e < n;
        hist_chunk<D>(h, valid ? (keyv[it] >> shift) & (BINS - 1) : (uint32_t)BINS, valid);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < BINS; b += kBlock) hist[hist_at<D>(b, tile, tiles, by_tile)] = h[b];
}

// One workgroup per digit: exclusive scan of that digit's tile counts.
__global__ __launch_bounds__(kBlock) void k_scan_digit(uint32_t *__restrict__ hist, uint32_t tiles,
                                                       uint32_t *__restrict__ totals)
{
    const uint32_t tot = block_scan_row<kBlock, 16>(hist + (size_t)blockIdx.x * tiles, tiles);
    if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// Scatter of one pass.  Each wavefront takes IT * 64 consecutive keys of the
// tile and counts its digits as it ranks them, without a barrier; the four
// counts of a digit then become its wavefronts' first places, and the keys
// are written.  (With a round of the whole workgroup and three barriers for
// every 256 keys: 8,000 keys of 9 bits 7.2 us, of 10 bits 13.1, the 810,448 of
// the column 11.0, 4 M of 10 bits 32; now 4.6, 5.3, 8.3 and 23.)
// Where the whole key is one digit, the scan of the digits is the bucket
// table: with `start`, the first tile writes it (buckets 0 .. nkeys).
template <int D, int IT>
__global__ __launch_bounds__(kBlock) void k_downsweep(const uint32_t *__restrict__ kin,
                                                      const uint32_t *__restrict__ vin,
                                                      uint32_t *__restrict__ kout,
                                                      uint32_t *__restrict__ vout, uint32_t n, int shift,
                                                      const uint32_t *__restrict__ hist, uint32_t tiles,
                                                      const uint32_t *__restrict__ totals, bool by_tile,
                                                      uint32_t *__restrict__ start, uint32_t nkeys)
{
    constexpr int BINS = 1 << D;
    constexpr int PT = BINS / kBlock;   // digits per thread in the bookkeeping
    static_assert(BINS % kBlock == 0, "digits must cover the block");
    constexpr int NW = kBlock / kWave;
    __shared__ uint32_t cnt[NW][BINS];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    // the tile's keys and values are read first: their loads overlap the
    // digit-base bookkeeping below and each other.  The tile order is that of
    // the histogram pass (same XCD for consecutive tiles, so the runs they
    // write side by side in each digit's range fill whole lines in one L2).
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t base = tile * (kBlock * IT) + (uint32_t)(wave * (IT * kWave) + lane);
    uint32_t keyv[IT], valv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const uint32_t e = base + it * kWave;
        keyv[it] = e < n ? kin[e] : 0u;
        valv[it] = e < n ? vin[e] : 0u;
    }
#pragma unroll
    for (int k = 0; k < BINS / kWave; ++k) cnt[wave][k * kWave + lane] = 0;
    // digit bases of this tile: exclusive scan of the digit totals (each
    // thread holds PT consecutive digits) plus the tile's offset in its digit
    uint32_t first[PT], mine[PT];
    uint32_t sum = 0;
    if (by_tile) {
        uint32_t all[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) all[k] = mine[k] = 0;
        const uint32_t *h = hist + tid * PT;
        constexpr uint32_t U = 32 / PT;   // tiles whose counts are in flight
        for (uint32_t t0 = 0; t0 < tiles; t0 += U) {
            uint32_t c[U][PT];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t t = t0 + u < tiles ? t0 + u : tiles - 1u;
#pragma unroll
                for (int k = 0; k < PT; ++k) c[u][k] = h[(size_t)t * BINS + k];
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < PT; ++k) {
                    all[k] += t0 + u < tiles ? c[u][k] : 0u;
                    mine[k] += t0 + u < tile ? c[u][k] : 0u;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            first[k] = sum;
            sum += all[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            first[k] = sum;
            sum += totals[tid * PT + k];
            mine[k] = hist[(size_t)(tid * PT + k) * tiles + tile];
        }
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan(sum, tot);
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const uint32_t d = (uint32_t)(tid * PT + k);
        first[k] += ex;
        if (start && tile == 0 && d <= nkeys) start[d] = first[k];
        if (start && tile == 0 && d + 1 == BINS && nkeys == BINS) start[BINS] = n;
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t rankv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const bool valid = base + it * kWave < n;
        const uint32_t d = (keyv[it] >> shift) & (BINS - 1);
        // Rank among the lanes of this wavefront with the same digit.  When the
        // valid lanes' digits do not decrease (the usual case: the keys arrive
        // nearly sorted), each digit is one run of lanes and the rank is the
        // distance from the run's first lane; otherwise one ballot per digit
        // bit gives each lane the mask of lanes holding its digit.
        const uint32_t prev = __shfl_up(d, 1, kWave);
        const uint64_t vmask = __ballot(valid);
        uint32_t rank, count;
        bool leader;
        if (__ballot(valid && lane > 0 && d < prev) == 0ull) {
            const bool head = valid && (lane == 0 || d != prev);
            const uint64_t heads = __ballot(head) | ~vmask;   // invalid lanes end the last run
            const uint64_t upto = heads & (lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1ull));
            const int from = 63 - __clzll((long long)upto);
            const uint64_t above = heads & ~(lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1ull));
            const int next = above ? __ffsll((unsigned long long)above) - 1 : kWave;
            rank = (uint32_t)(lane - from);
            count = (uint32_t)(next - from);
            leader = valid && next == lane + 1;
        } else {
            uint64_t mask = vmask;
#pragma unroll
            for (int b = 0; b < D; ++b) {
                bool bit = (d >> b) & 1u;
                uint64_t bm = __ballot(bit);
                mask &= bit ? bm : ~bm;
            }
            rank = (uint32_t)__popcll(mask & below);
            count = (uint32_t)__popcll(mask);
            leader = valid && ((mask >> lane) == 1ull);
        }
        const uint32_t seen = valid ? cnt[wave][d] : 0u;   // by this wavefront, so far
        wave_lds_order();
        if (leader) cnt[wave][d] = seen + count;
        wave_lds_order();
        rankv[it] = seen + rank;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        uint32_t at = first[k] + mine[k];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t c = cnt[w][tid * PT + k];
            cnt[w][tid * PT + k] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        if (base + it * kWave < n) {
            const uint32_t pos = cnt[wave][(keyv[it] >> shift) & (BINS - 1)] + rankv[it];
            kout[pos] = keyv[it];
            vout[pos] = valv[it];
        }
    }
}

// How a sort of n keys below nkeys goes: digits of D bits, in tiles of
// kBlock * items keys.  While a tile's workgroup can read every tile's counts
// (64 KB at most) the scatter adds them up itself, 32 loads in flight, and the
// scan's launch (3.6 to 4.6 us a pass) is saved: up to 131,072 keys of 8-bit
// digits, 65,536 of wider ones (there a 100,000-key pass takes 7.1 us, and 7.2
// with a scan beside it; beyond, the counts read grow with the square of n).
// Up to 32,768 keys the tiles are also a quarter or half as long, so that more
// workgroups share the work (the workspace holds n / 2 counts).
struct SortPlan {
    int D, passes, items;
    uint32_t tiles;
    bool by_tile;
};

inline int key_bits(uint32_t nkeys);
inline int radix_digit_bits(uint32_t nkeys);
template <int D>
constexpr int few_items = 1 << (D - 7);   // 2, 4, 8

inline SortPlan sort_plan(uint32_t n, uint32_t nkeys)
{
    SortPlan p;
    const int bits = key_bits(nkeys);
    p.passes = bits > 0 ? (bits + kMaxRadixBits - 1) / kMaxRadixBits : 1;
    p.D = radix_digit_bits(nkeys);
    const uint32_t most = 16384u >> p.D;   // tiles of 64 KB of counts
    p.items = p.D == 8 ? few_items<8> : p.D == 9 ? few_items<9> : few_items<10>;
    p.tiles = div_up(n, (uint64_t)kBlock * p.items);
    if (p.tiles > most) {
        p.items = p.D == 10 ? sort_items<10> : sort_items<9>;
        p.tiles = div_up(n, (uint64_t)kBlock * p.items);
    }
    p.by_tile = p.tiles <= most;
    return p;
}

// One LSD pass with D-bit digits starting at bit `shift`; with hist_ready the
// per-tile digit counts are already in ws.hist (written by the kernel that
// produced the keys, over the same tiles).  With `start`, also the bucket
// table of a sort of one pass.
template <int D, int IT>
void sort_pass(const Workspace &ws, const SortPlan &p, uint32_t n, int shift, int cur, hipStream_t s,
               bool hist_ready, uint32_t *start, uint32_t nkeys)
{
    if (!hist_ready) k_upsweep<D, IT><<<p.tiles, kBlock, 0, s>>>(ws.keys[cur], n, shift, ws.hist, p.tiles, p.by_tile);
    if (!p.by_tile) k_scan_digit<<<1u << D, kBlock, 0, s>>>(ws.hist, p.tiles, ws.totals);
    k_downsweep<D, IT><<<p.tiles, kBlock, 0, s>>>(ws.keys[cur], ws.vals[cur], ws.keys[cur ^ 1], ws.vals[cur ^ 1], n,
                                                  shift, ws.hist, p.tiles, ws.totals, p.by_tile, start, nkeys);
}

// Number of bits needed for keys below nkeys.
inline int key_bits(uint32_t nkeys)
{
    int b = 0;
    while (b < 32 && (uint64_t(1) << b) < nkeys) ++b;
    return b;
}

// Digit width (8 to 10 bits) of a sort of keys below nkeys, in as few passes
// as possible.
inline int radix_digit_bits(uint32_t nkeys)
{
    const int bits = key_bits(nkeys);
    const int passes = bits > 0 ? (bits + kMaxRadixBits - 1) / kMaxRadixBits : 1;
    const int dbits = (bits + passes - 1) / passes;
    return dbits < 8 ? 8 : dbits;
}

// Sorts (ws.keys[0], ws.vals[0]) of n entries, keys below nkeys; returns the
// index of the key/value buffer pair that holds the result.  With
// first_hist, the first pass's per-tile digit counts are already in ws.hist.
// A sort of one pass also writes the bucket table to `start`, if given.
inline int radix_sort(const Workspace &ws, uint32_t n, uint32_t nkeys, hipStream_t s, bool first_hist = false,
                      uint32_t *start = nullptr)
{
    const SortPlan p = sort_plan(n, nkeys);
    if (p.passes > 1) start = nullptr;
    int cur = 0;
    for (int ps = 0; ps < p.passes; ++ps) {
        const int shift = ps * p.D;
        const bool ready = first_hist && ps == 0;
        if (p.D == 8 && p.items == few_items<8>)
            sort_pass<8, few_items<8>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        else if (p.D == 8)
            sort_pass<8, sort_items<8>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        else if (p.D == 9 && p.items == few_items<9>)
            sort_pass<9, few_items<9>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        else if (p.D == 9)
            sort_pass<9, sort_items<9>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        else if (p.items == few_items<10>)
            sort_pass<10, few_items<10>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        else
            sort_pass<10, sort_items<10>>(ws, p, n, shift, cur, s, ready, start, nkeys);
        cur ^= 1;
    }
    return cur;
}

}  // namespace

}  // namespace sph
