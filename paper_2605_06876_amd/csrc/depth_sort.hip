// Depth order of the entries: a sample sort whose buckets are finished in LDS.
//
// The entries are sorted stably by the float bits of their depth (entry ids
// ascending on ties) and the tile counts scanned in that order.  As an LSD
// radix sort that is four digit passes of three launches and two launches of
// the scan, most of them launch latency below a few hundred thousand
// entries, and every entry moved four times through memory above.  Here:
//   up      every block takes NB - 1 splitters from the same sample of the
//           keys, then counts its tile's keys per bucket
//           (bucket = splitters <= key, so equal keys share a bucket);
//   scan    (above DS_ROWS tiles) the counts' prefixes over the tiles; below,
//           each block of the next launch sums the tiles' rows itself;
//   down    keys scattered by bucket, in entry order within a bucket, and the
//           tile counts summed per bucket;
//   local   one block per bucket: its keys placed by counting (cell_places) or,
//           where they are too uneven for that, sorted by digit passes, in
//           registers and LDS or in global memory; then the entries, their tile counts and the
//           counts' exclusive prefix written once.
// A sort of up to DS_ONE entries is the local step alone, one launch.
// Radix sort and scan against this (us, MI355X): 2,000 entries 50 -> 9, 20,000
// 65 -> 22, 150,000 80 -> 36, 600,000 96 -> 52, 1,000,000 99 -> 69.  What bounds it
// now: small sorts three launches and their barriers; large ones the LDS pipe
// of the CU with the fullest bucket.
//
// Buckets follow the keys' distribution (the splitters are quantiles of the
// sample), except that equal keys cannot be told apart by splitters.  A depth that
// more than one splitter falls on gets a bucket of its own, which needs no sorting
// and which the blocks of the buckets left empty write with its own (splitters,
// share_bucket).  Left to be sorted in global memory by one block are buckets of few
// depths above 4 T keys, or above the LDS capacity (two or three depths with a
// 200th of a million entries each).
// Depth order, scan and pair sort of 1,048,576 entries (us; in brackets with one
// block for every bucket, then with the radix sort): spread depths 110 (110, 141), all
// equal 103 (1467, 132), nine in ten equal 122 (3063, 136), 160 depths 174 (468, 139),
// two clouds' entries in turn 155 (3894, 140), a third of the entries behind the camera
// 103 (317, 128).
// Values are the entry ids, so the first scatter reads only keys, straight
// from the projection's depth keys.
#include <type_traits>

#include "internal.h"

namespace {

constexpr int DT = 1024;                 // threads of a block
constexpr int DW = DT / 64;
constexpr int NB = 256;                  // buckets: a block for each of the 256 CUs to finish
// Where the forms change (us for the whole sort, 640x480 view):
//   one block     1,000: 6.6, 2,000: 8.5, 4,096: 15.6, 6,000: 23; three launches take 19 from there up
//   256 threads   a bucket, 100,000: 12 for the buckets (1024 threads: 14); 200,000: 22 (14)
//   tiles of 2048 and a sample of 1024: 524,000: 47; of 4096 and 2048 (fewer, fuller buckets over
//                 the capacity): 525,000: 49
//   four launches 1,000,000: 70, 1,300,000: 87; the radix sort and scan 1,400,000: 114 (at more
//                 entries the buckets outgrow LDS)
constexpr int64_t DS_ONE = 4096;         // entries sorted by one block
constexpr int64_t DS_SMALL = 1 << 19;    // entries up to which tiles hold 2048 keys and the sample 1024, above 4096 and 2048
constexpr int64_t DS_LIGHT = 1 << 17;    // entries up to which a bucket's block has 256 threads, above 1024
constexpr int DS_ITEMS = 16;             // keys per thread of the largest bucket sorted in LDS (16,384)
constexpr int DS_ROWS = 64;              // tiles whose counts the scatter sums itself
constexpr int SLOW_ITEMS = 4;            // keys per thread and step of the global-memory path

// Workspace words: splitters, bucket totals, tile-count sums, then per tile the
// counts and, of the buckets of one depth, (keys, their tile counts' sum).
struct DsWs {
    uint32_t *split, *total, *ntsum, *counts;
    uint2 *part;
};
DsWs ds_ws(void *ws, int64_t tiles) {
    uint32_t *p = reinterpret_cast<uint32_t *>(ws);
    return DsWs{p, p + NB, p + 2 * NB, p + 3 * NB, reinterpret_cast<uint2 *>(p + 3 * NB + tiles * NB)};
}

// A depth's key, from the least depth kept (AS_NEAR, rounded to float) on.  The projection
// keeps nothing nearer or behind, so those entries' order shows in nothing (they touch no
// tile): they take one key above all others.  With their own bits, which span both
// signs and all exponents down to zero, they would stretch the range of the buckets
// at both ends, whose cells then hold too many keys.  (Infinity and NaN stay below CULLED.)
constexpr uint32_t KEY_LEAST = __builtin_bit_cast(uint32_t, (float)AS_NEAR), CULLED = 0x80000000u - KEY_LEAST;
__device__ __forceinline__ uint32_t live_key(uint32_t depth_bits) { return min(depth_bits - KEY_LEAST, CULLED); }

// f(0), f(1), .. f(N - 1) with compile-time indices: the per-thread arrays
// below are then registers from the start (as loops to be unrolled, those of
// 16 elements were kept as memory, or as whole vectors copied at each store).
template <int N, typename F>
__device__ __forceinline__ void each(F f) {
    if constexpr (N > 0) {
        each<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Exclusive scan of one value per thread over the block; *sum gets the total.
// s_w: a word per wave (NW); a barrier before its first write.
template <int NW = DW>
__device__ __forceinline__ uint32_t scan_block(uint32_t v, uint32_t *s_w, uint32_t *sum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t inc = wave_prefix(v);
    __syncthreads();
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t pre = 0, all = 0;
#pragma unroll
    for (int k = 0; k < NW; k++) {
        const uint32_t x = s_w[k];
        if (k < w) pre += x;
        all += x;
    }
    *sum = all;
    return pre + inc - v;
}

// Least and greatest of the block's keys (T threads; sm, sx a word per wave).
template <int T>
__device__ __forceinline__ void block_range(uint32_t mn, uint32_t mx, uint32_t *sm, uint32_t *sx, uint32_t *lo,
                                            uint32_t *hi) {
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor((int)mn, o, 64));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = mn;
        sx[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    for (int k = 0; k < T / 64; k++) {
        mn = min(mn, sm[k]);
        mx = max(mx, sx[k]);
    }
    *lo = mn;
    *hi = mx;
}

// Placing keys by counting: SB cells divide the keys' range, a key's
// place is the first of its cell plus its rank in the cell, by (key, index)
// against the few others there.  The cells are even over the range, or, for
// the nearest and the deepest bucket, which hold the tails of the distribution, of
// widths growing from the range's dense end (CELLS_FROM_HI, CELLS_FROM_LO: SB / 32
// cells per octave of the distance to it).  No digit passes and no ballots: four barriers
// apart from the scan of the cells.  Where a cell holds more than CELL_MAX keys
// (many equal keys, or a range stretched by outliers) nothing is placed
// and false returned, to the whole block: the caller takes the digit passes.
// With CULL, keys may be CULLED: those are placed after the others, in any order (a
// bucket's keys are not: they have one of their own).
constexpr uint32_t CELL_MAX = 64;

enum CellMap { CELLS_EVEN, CELLS_FROM_HI, CELLS_FROM_LO };

template <int SB>
__device__ __forceinline__ uint32_t octave_cell(uint32_t x) {
    constexpr int F = __builtin_ctz(SB) - 5;
    const int e = 31 - __clz(x | 1);
    return e < F ? x : ((uint32_t)(e - F + 1) << F) + ((x >> (e - F)) & ((1u << F) - 1u));   // < SB
}

template <int SB>
__device__ __forceinline__ uint32_t cell_of(uint32_t key, uint32_t lo, uint32_t hi, int shift, CellMap map) {
    if (map == CELLS_FROM_HI) return (uint32_t)SB - 1u - octave_cell<SB>(hi - key);
    if (map == CELLS_FROM_LO) return octave_cell<SB>(key - lo);
    return (key - lo) >> shift;
}

template <int T, int CAP, int SB>
struct CellShared {
    uint32_t cell[SB + 1];
    uint32_t key[CAP];
    uint16_t idx[CAP];
    uint32_t w[T / 64], mn[T / 64], mx[T / 64], culled;
};

// Element j of thread t is index i0 + stride j (valid below m).
template <int T, int ITEMS, int CAP, int SB, bool CULL>
__device__ __forceinline__ bool cell_places(const uint32_t (&key)[ITEMS], uint32_t i0, uint32_t stride, uint32_t m,
                                            CellMap map, CellShared<T, CAP, SB> &sh, uint32_t (&place)[ITEMS]) {
    constexpr int PER = SB / T;
    const int tid = threadIdx.x;
    auto valid = [&](int j) { return i0 + (uint32_t)j * stride < m; };
    auto ok = [&](int j) { return valid(j) && (!CULL || key[j] != CULLED); };
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) {
            lo = min(lo, key[j]);
            hi = max(hi, key[j]);
        }
    });
#pragma unroll
    for (int k = 0; k < PER; k++) sh.cell[tid + k * T] = 0u;
    if (CULL && tid == 0) sh.culled = 0u;
    block_range<T>(lo, hi, sh.mn, sh.mx, &lo, &hi);   // (its barrier: the cells are clear)
    const int bits = hi > lo ? 32 - __clz(hi - lo) : 0;
    const int shift = bits > __builtin_ctz(SB) ? bits - __builtin_ctz(SB) : 0;
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) place[j] = atomicAdd(&sh.cell[cell_of<SB>(key[j], lo, hi, shift, map)], 1u);
    });
    __syncthreads();
    uint32_t c[PER], sum = 0, most = 0, all;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        c[k] = sh.cell[PER * tid + k];
        sum += c[k];
        most = max(most, c[k]);
    }
    for (int o = 32; o > 0; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
    if ((tid & 63) == 0) sh.mx[tid >> 6] = most;
    uint32_t run = scan_block<T / 64>(sum, sh.w, &all);   // (its barriers: mx is whole)
    for (int k = 0; k < T / 64; k++) most = max(most, sh.mx[k]);
    if (most > CELL_MAX) return false;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        sh.cell[PER * tid + k] = run;
        run += c[k];
    }
    if (tid == T - 1) sh.cell[SB] = run;
    if (CULL)
        each<ITEMS>([&](auto J) {   // (all: the keys that are not culled)
            constexpr int j = J;
            const bool cull = valid(j) && key[j] == CULLED;
            const uint64_t bal = __builtin_amdgcn_ballot_w64(cull);
            if (bal) {
                uint32_t first = 0;
                if ((tid & 63) == 0) first = atomicAdd(&sh.culled, (uint32_t)__popcll(bal));
                first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
                if (cull) place[j] = all + first + (uint32_t)__popcll(bal & lanemask_lt());
            }
        });
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) {
            const uint32_t p = sh.cell[cell_of<SB>(key[j], lo, hi, shift, map)] + place[j];
            sh.key[p] = key[j];
            sh.idx[p] = (uint16_t)(i0 + (uint32_t)j * stride);
        }
    });
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) {
            const uint32_t cl = cell_of<SB>(key[j], lo, hi, shift, map), beg = sh.cell[cl], end = sh.cell[cl + 1];
            const uint32_t i = i0 + (uint32_t)j * stride;
            uint32_t r = beg;
            for (uint32_t q = beg; q < end; q++) {
                const uint32_t k = sh.key[q];
                bool ahead = k < key[j];
                if (k == key[j]) ahead = sh.idx[q] < i;   // mostly the key itself
                r += ahead ? 1u : 0u;
            }
            place[j] = r;
        }
    });
    return true;
}

// The block's I * 1024 keys ascending, key j of thread t at j * 1024 + t (bitonic:
// strides below a wave by lane exchange, up to the block through LDS, s: I * 1024
// words, the last one between a thread's two).
template <int I>
__device__ __forceinline__ void bitonic_block(uint32_t (&v)[I], uint32_t *s) {
    static_assert(I <= 2, "at most two keys a thread");
    const int tid = threadIdx.x;
    for (int k = 2; k <= I * DT; k <<= 1)
        for (int st = k >> 1; st > 0; st >>= 1) {
            if (st >= DT) {
                const uint32_t a = v[0], b = v[I - 1];
                v[0] = min(a, b);
                v[I - 1] = max(a, b);
                continue;
            }
            if (st >= 64) {
                __syncthreads();
#pragma unroll
                for (int j = 0; j < I; j++) s[j * DT + tid] = v[j];
                __syncthreads();
            }
#pragma unroll
            for (int j = 0; j < I; j++) {
                const uint32_t o = st < 64 ? (uint32_t)__shfl_xor((int)v[j], st, 64) : s[j * DT + (tid ^ st)];
                const bool lower = (tid & st) == 0, up = ((j * DT + tid) & k) == 0;
                v[j] = lower == up ? min(v[j], o) : max(v[j], o);
            }
        }
}

// Where sample k of S is taken: somewhere in the k-th of S equal parts of the
// entries.  Always in the middle, it would be every 2^m-th entry of most sets, and see
// one kind of entries where kinds alternate.
template <int S>
__device__ __forceinline__ uint32_t sample_at(uint32_t k, uint32_t n) {
    static_assert((int64_t)S * DEPTH_SORT_MAX <= 0xFFFFFFFFll, "products of 32 bits");
    const uint32_t lo = k * n / S, hi = (k + 1) * n / S;
    uint32_t h = (k + 1) * 0x9E3779B1u;
    h = (h ^ (h >> 15)) * 0x85EBCA77u;
    return lo + __umulhi(h, hi - lo);
}

// NB - 1 splitters from a sample of S keys, into s_split: NB - 3 quantiles of it, and
// the last two around CULLED, which thus has the last bucket but one (the last
// is empty).  The sample is placed by cells, a skewed one (see cell_places) sorted.
//
// Where splitters are equal, a depth holds more than about one in 128 of the
// entries.  Of a run of equal splitters the last is raised by one: the bucket
// before it then holds that depth alone, in order as it stands, and the buckets of the
// run before that one are empty, in number as the share of the entries it holds,
// so their blocks can write it between them (share_bucket).
// (To be seen by other threads after the caller's next barrier.)
template <int S>
__device__ __forceinline__ void splitters(const uint32_t *__restrict__ keys, int64_t n, CellShared<DT, S, 2 * DT> &sh,
                                          uint32_t *s_split) {
    constexpr int I = S / DT;
    const int tid = threadIdx.x;
    uint32_t v[I], place[I];
#pragma unroll
    for (int j = 0; j < I; j++) v[j] = live_key(keys[sample_at<S>((uint32_t)(tid + j * DT), (uint32_t)n)]);
    if (!cell_places<DT, I, S, 2 * DT, true>(v, (uint32_t)tid, DT, (uint32_t)S, CELLS_EVEN, sh, place)) {
        __syncthreads();
        bitonic_block<I>(v, sh.key);
        each<I>([&](auto J) {
            constexpr int j = J;
            place[j] = (uint32_t)(j * DT + tid);
        });
    }
    each<I>([&](auto J) {   // places k S / (NB - 2), k = 1 .. NB - 3, rounded up
        constexpr int j = J;
        const uint32_t k = place[j] * (NB - 2) / S;
        if (place[j] > 0 && k != (place[j] - 1) * (NB - 2) / S) s_split[k - 1] = v[j];
    });
    if (tid < 2) s_split[NB - 3 + tid] = CULLED + (uint32_t)tid;
    __syncthreads();
    const uint32_t x = tid < NB - 1 ? s_split[tid] : 0u;
    const bool raise = tid > 0 && tid < NB - 3 && s_split[tid - 1] == x && s_split[tid + 1] != x && x < CULLED;
    __syncthreads();
    if (raise) s_split[tid] = x + 1;
}

// Whether bucket b (one of 1 .. NB - 2) holds one depth at most, between its splitters.
__device__ __forceinline__ bool one_depth(const uint32_t *split, int b) { return split[b] - split[b - 1] <= 1u; }

// Ranks a wave's keys among equal digits, in order: loc[j] is the number of
// the wave's keys of digit dig(j) before key j among those with ok(j); cnt[]
// gets the wave's counts.  Digits have at most NBITS bits.
template <int ITEMS, int NBITS, typename Dig, typename Ok>
__device__ __forceinline__ void rank_wave(uint32_t *cnt, uint32_t (&loc)[ITEMS], Dig dig, Ok ok) {
    const uint64_t lt = lanemask_lt();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        uint32_t d = dig(j);
        // one key's ballots at a time: taken all at once they fill the registers
        __asm__ __volatile__("" : "+v"(d) : : "memory");
        const bool use = ok(j);
        uint64_t peers = __ballot(use);
#pragma unroll
        for (int bit = 0; bit < NBITS; bit++) {
            const bool set = (d >> bit) & 1u;
            const uint64_t m = __ballot(set);
            peers &= set ? m : ~m;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t before = cnt[d];
        __builtin_amdgcn_wave_barrier();
        if (use && rank == 0) cnt[d] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        loc[j] = before + rank;
    });
}

// ---- up: splitters and counts ---------------------------------------------------------

__device__ __forceinline__ uint32_t bucket_of(const uint32_t *s_split, uint32_t key) {
    uint32_t b = 0;
#pragma unroll
    for (int step = NB / 2; step > 0; step >>= 1)
        if (s_split[b + step - 1] <= key) b += step;
    return b;
}

// Bucket counts per tile of DT * R keys; rows (counts[tile][NB]) or columns
// (counts[NB][tile]).  Each block takes the splitters from the same sample
// itself (a launch of its own would cost more); block 0 keeps them for the scatter.
template <int R, int S>
__global__ void __launch_bounds__(DT) k_ds_up(const uint32_t *__restrict__ keys, int64_t n, DsWs ws, int64_t tiles,
                                              int rows) {
    __shared__ uint32_t s_split[NB];
    __shared__ uint32_t s_h[2][NB];
    __shared__ CellShared<DT, S, 2 * DT> s_cells;
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x, base = tile * (DT * R);
    uint32_t key[R];
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int64_t i = base + j * DT + tid;
        key[j] = i < n ? live_key(keys[i]) : 0u;
    }
    splitters<S>(keys, n, s_cells, s_split);
    if (tile == 0 && tid < NB - 1) ws.split[tid] = s_split[tid];
    for (int i = tid; i < 2 * NB; i += DT) (&s_h[0][0])[i] = 0u;
    if (tile == 0)
        for (int i = tid; i < NB; i += DT) ws.ntsum[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < R; j++)
        if (base + j * DT + tid < n) atomicAdd(&s_h[tid & 1][bucket_of(s_split, key[j])], 1u);
    __syncthreads();
    for (int d = tid; d < NB; d += DT) {
        const uint32_t c = s_h[0][d] + s_h[1][d];
        if (rows) ws.counts[tile * NB + d] = c;
        else ws.counts[(int64_t)d * tiles + tile] = c;
    }
}

// One block per bucket: the column's exclusive prefix over the tiles, in
// place, and its total.
__global__ void __launch_bounds__(256) k_ds_scan(DsWs ws, int64_t tiles) {
    __shared__ uint32_t s_w[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t *col = ws.counts + (int64_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    for (int64_t t0 = 0; t0 < tiles; t0 += 1024) {
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int64_t t = t0 + 4 * tid + k;
            v[k] = t < tiles ? col[t] : 0u;
            sum += v[k];
        }
        uint32_t inc = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = (uint32_t)__shfl_up((int)inc, o, 64);
            if (lane >= o) inc += x;
        }
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        uint32_t run = carry + inc - sum;
        for (int k = 0; k < 4; k++) {
            if (k < w) run += s_w[k];
            carry += s_w[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int64_t t = t0 + 4 * tid + k;
            if (t < tiles) col[t] = run;
            run += v[k];
        }
    }
    if (tid == 0) ws.total[blockIdx.x] = carry;
}

// ---- down: scatter by bucket -------------------------------------------------------------

template <int R>
__global__ void __launch_bounds__(DT) k_ds_down(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ nt,
                                                int64_t n, DsWs ws, int64_t tiles, int rows,
                                                uint32_t *__restrict__ kout, uint32_t *__restrict__ vout) {
    static_assert(NB == 256, "bucket ids of eight bits");
    constexpr int TILE = DT * R;
    __shared__ uint32_t s_split[NB];
    __shared__ uint32_t s_wcnt[DW][NB];
    __shared__ uint32_t s_boff[NB], s_gdst[NB], s_nt[NB];
    __shared__ uint32_t s_w[DW];
    __shared__ uint32_t s_key[TILE], s_val[TILE];
    __shared__ uint8_t s_bkt[TILE];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t tile = blockIdx.x, base = tile * TILE;
    const int cnt = n - base < TILE ? (int)(n - base) : TILE;
    uint32_t key[R], d[R], loc[R], cn[R];
    auto ok = [&](int j) { return w * (64 * R) + j * 64 + lane < cnt; };
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int i = w * (64 * R) + j * 64 + lane;
        key[j] = ok(j) ? live_key(keys[base + i]) : 0u;
        cn[j] = nt && ok(j) ? nt[base + i] : 0u;
    }
    // the tile's offset in each bucket and the bucket totals
    uint32_t before = 0, total = 0;
    if (rows) {
        // DT / NB threads a bucket, each every (DT / NB)-th row
        constexpr int Q = DT / NB;
        const int b = tid % NB, q = tid / NB;
#pragma unroll 4
        for (int64_t t = q; t < tiles; t += Q) {
            const uint32_t c = ws.counts[t * NB + b];
            if (t < tile) before += c;
            total += c;
        }
        // fold the quarters through the (not yet used) reorder buffers
        s_key[q * NB + b] = before;
        s_val[q * NB + b] = total;
        __syncthreads();
        before = total = 0;
        if (tid < NB)
            for (int k = 0; k < Q; k++) {
                before += s_key[k * NB + tid];
                total += s_val[k * NB + tid];
            }
        if (tile == 0 && tid < NB) ws.total[tid] = total;
    } else if (tid < NB) {
        before = ws.counts[(int64_t)tid * tiles + tile];
        total = ws.total[tid];
    }
    if (tid < NB - 1) s_split[tid] = ws.split[tid];
    for (int i = tid; i < DW * NB; i += DT) (&s_wcnt[0][0])[i] = 0u;
    for (int i = tid; i < NB; i += DT) s_nt[i] = 0u;
    uint32_t sum;
    const uint32_t gstart = scan_block(tid < NB ? total : 0u, s_w, &sum);
#pragma unroll
    for (int j = 0; j < R; j++) {
        d[j] = bucket_of(s_split, key[j]);
        if (cn[j]) atomicAdd(&s_nt[d[j]], cn[j]);
    }
    rank_wave<R, 8>(s_wcnt[w], loc, [&](int j) { return d[j]; }, ok);
    __syncthreads();
    uint32_t tot = 0;
    if (tid < NB) {
#pragma unroll
        for (int k = 0; k < DW; k++) {
            const uint32_t c = s_wcnt[k][tid];
            s_wcnt[k][tid] = tot;
            tot += c;
        }
        if (s_nt[tid]) atomicAdd(&ws.ntsum[tid], s_nt[tid]);
        if (nt && tid > 0 && tid < NB - 1 && one_depth(s_split, tid)) ws.part[tile * NB + tid] = make_uint2(tot, s_nt[tid]);
    }
    const uint32_t boff = scan_block(tot, s_w, &sum);
    if (tid < NB) {
        s_boff[tid] = boff;
        s_gdst[tid] = gstart + before - boff;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < R; j++)
        if (ok(j)) {
            const uint32_t lp = s_boff[d[j]] + s_wcnt[w][d[j]] + loc[j];
            s_key[lp] = key[j];
            s_val[lp] = (uint32_t)(base + w * (64 * R) + j * 64 + lane);
            s_bkt[lp] = (uint8_t)d[j];
        }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int i = j * DT + tid;
        if (i < cnt) {
            const uint32_t g = s_gdst[s_bkt[i]] + (uint32_t)i;
            kout[g] = s_key[i];
            vout[g] = s_val[i];
        }
    }
}

// ---- local: buckets finished in LDS ---------------------------------------------------

// T threads
template <int T>
struct LocalShared {
    static constexpr int NW = T / 64;
    uint32_t wcnt[NW][256];
    uint32_t boff[256], run[256];
    uint32_t w[NW], mn[NW], mx[NW];
};

// One stable digit pass over the block's keys: thread element j is index
// w (64 ITEMS) + 64 j + lane of m; buf holds at least m words.
template <int T, int ITEMS>
__device__ __forceinline__ void local_pass(uint32_t (&key)[ITEMS], uint32_t (&val)[ITEMS], int m, uint32_t lowest,
                                           int shift, uint32_t mask, LocalShared<T> &sh, uint32_t *buf) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    auto ok = [&](int j) { return w * (64 * ITEMS) + j * 64 + lane < m; };
    auto dig = [&](int j) { return ((key[j] - lowest) >> shift) & mask; };
    for (int i = tid; i < T / 64 * 256; i += T) (&sh.wcnt[0][0])[i] = 0u;
    __syncthreads();
    uint32_t loc[ITEMS];
    rank_wave<ITEMS, 8>(sh.wcnt[w], loc, dig, ok);
    __syncthreads();
    uint32_t tot = 0, sum;
    if (tid < 256) {
#pragma unroll
        for (int k = 0; k < T / 64; k++) {
            const uint32_t c = sh.wcnt[k][tid];
            sh.wcnt[k][tid] = tot;
            tot += c;
        }
    }
    const uint32_t boff = scan_block<T / 64>(tot, sh.w, &sum);
    if (tid < 256) sh.boff[tid] = boff;
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        const uint32_t d = dig(j);
        loc[j] += sh.boff[d] + sh.wcnt[w][d];
        if (ok(j)) buf[loc[j]] = key[j];
    });
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) key[j] = buf[w * (64 * ITEMS) + j * 64 + lane];
    });
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) buf[loc[j]] = val[j];
    });
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if (ok(j)) val[j] = buf[w * (64 * ITEMS) + j * 64 + lane];
    });
}

// Digits of the bits in which keys of this range differ.
__device__ __forceinline__ void digits_of(uint32_t lo, uint32_t hi, int *passes, int *nbits) {
    const int bits = hi > lo ? 32 - __clz(hi - lo) : 0;
    *passes = (bits + 7) / 8;
    *nbits = *passes ? (bits + *passes - 1) / *passes : 0;
}

// The sorted bucket's entries, tile counts and their exclusive prefix
// from base: element j of a thread is index w (64 ITEMS) + 64 j + lane.
// Returns the prefix after the last.
template <int T, int ITEMS>
__device__ __forceinline__ uint32_t write_bucket(const uint32_t (&val)[ITEMS], uint32_t (&cn)[ITEMS], uint32_t m,
                                             uint32_t base, uint32_t *s_w, uint32_t *__restrict__ order,
                                             uint32_t *__restrict__ nt_sorted, uint32_t *__restrict__ offsets) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t i0 = (uint32_t)(w * (64 * ITEMS) + lane);
    if (!nt_sorted) {   // the order alone
        each<ITEMS>([&](auto J) {
            constexpr int j = J;
            if (i0 + j * 64 < m) order[i0 + j * 64] = val[j];
        });
        return base;
    }
    uint32_t sum = 0;
    each<ITEMS>([&](auto J) { sum += cn[J]; });
    sum = wave_prefix(sum);
    __syncthreads();
    if (lane == 63) s_w[w] = sum;
    __syncthreads();
    uint32_t end = base;
    for (int k = 0; k < T / 64; k++) {
        end += s_w[k];
        if (k < w) base += s_w[k];
    }
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        const uint32_t inc = wave_prefix(cn[j]);
        const uint32_t i = i0 + j * 64;
        if (i < m) {
            order[i] = val[j];
            nt_sorted[i] = cn[j];
            offsets[i] = base + inc - cn[j];
        }
        base += last_lane(inc);
    });
    return end;
}

// A bucket of m <= T * ITEMS keys (kin, vin: its first; vin NULL: the ids are
// the positions) placed by cells; false when they are too skewed for that.
template <int T, int ITEMS, int CAP, int SB, bool CULL>
__device__ __forceinline__ bool cell_sort(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint32_t m,
                                          uint32_t base, const uint32_t *__restrict__ nt, uint32_t *__restrict__ order,
                                          uint32_t *__restrict__ nt_sorted, uint32_t *__restrict__ offsets, CellMap map,
                                          CellShared<T, CAP, SB> &sh) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t key[ITEMS], val[ITEMS], place[ITEMS];
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        const uint32_t i = (uint32_t)(tid + j * T);
        key[j] = val[j] = 0u;
        if (i < m) {
            key[j] = CULL ? live_key(kin[i]) : kin[i];
            val[j] = vin ? vin[i] : i;
        }
    });
    if (!cell_places<T, ITEMS, CAP, SB, CULL>(key, (uint32_t)tid, T, m, map, sh, place)) return false;
    // into sorted order through the cells' keys, which are read
    const uint32_t i0 = (uint32_t)(w * (64 * ITEMS) + lane);
    __syncthreads();
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        if ((uint32_t)(tid + j * T) < m) sh.key[place[j]] = val[j];
    });
    __syncthreads();
    each<ITEMS>([&](auto J) {   // (key[] is free for the tile counts)
        constexpr int j = J;
        const bool in = i0 + j * 64 < m;
        val[j] = in ? sh.key[i0 + j * 64] : 0u;
        key[j] = nt && in ? nt[val[j]] : 0u;
    });
    write_bucket<T, ITEMS>(val, key, m, base, sh.w, order, nt_sorted, offsets);
    return true;
}

// The same by digit passes in registers and LDS, whatever the distribution.
template <int T, int ITEMS, bool RAW = false>
__device__ __forceinline__ void local_sort(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint32_t m,
                                           uint32_t base, const uint32_t *__restrict__ nt, uint32_t *__restrict__ order,
                                           uint32_t *__restrict__ nt_sorted, uint32_t *__restrict__ offsets,
                                           LocalShared<T> &sh, uint32_t *buf) {
    const uint32_t i0 = (threadIdx.x >> 6) * (64 * ITEMS) + (threadIdx.x & 63);
    uint32_t key[ITEMS], val[ITEMS];
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    each<ITEMS>([&](auto J) {
        constexpr int j = J;
        const uint32_t i = i0 + j * 64;
        key[j] = val[j] = 0u;
        if (i < m) {
            key[j] = RAW ? live_key(kin[i]) : kin[i];
            val[j] = vin ? vin[i] : i;
            mn = min(mn, key[j]);
            mx = max(mx, key[j]);
        }
    });
    uint32_t lo, hi;
    __syncthreads();
    block_range<T>(mn, mx, sh.mn, sh.mx, &lo, &hi);
    int passes, nbits;
    digits_of(lo, hi, &passes, &nbits);
    for (int p = 0; p < passes; p++) local_pass<T, ITEMS>(key, val, (int)m, lo, p * nbits, (1u << nbits) - 1u, sh, buf);
    each<ITEMS>([&](auto J) {   // (key[] is free for the tile counts)
        constexpr int j = J;
        key[j] = nt && i0 + j * 64 < m ? nt[val[j]] : 0u;
    });
    write_bucket<T, ITEMS>(val, key, m, base, sh.w, order, nt_sorted, offsets);
}

// A bucket of any size, in global memory: LSD passes between the two buffers
// by this block alone, the result's entries written to order (= v0).
template <int T>
__device__ __attribute__((noinline)) void slow_sort(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, int64_t start, int64_t m,
                          uint32_t base, const uint32_t *__restrict__ nt, uint32_t *__restrict__ nt_sorted,
                          uint32_t *__restrict__ offsets, LocalShared<T> &sh) {
    constexpr int STEP = T * SLOW_ITEMS;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t *ks = k1 + start, *vs = v1 + start, *kd = k0 + start, *vd = v0 + start;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    for (int64_t i = tid; i < m; i += T) {
        mn = min(mn, ks[i]);
        mx = max(mx, ks[i]);
    }
    uint32_t lo, hi, sum;
    block_range<T>(mn, mx, sh.mn, sh.mx, &lo, &hi);
    int passes, nbits;
    digits_of(lo, hi, &passes, &nbits);
    const uint32_t mask = (1u << nbits) - 1u;
    for (int p = 0; p < passes; p++) {
        const int shift = p * nbits;   // (< 32: the passes cover at most 32 bits)
        __syncthreads();
        if (tid < 256) sh.boff[tid] = 0u;
        __syncthreads();
        for (int64_t i = tid; i < m; i += T) atomicAdd(&sh.boff[((ks[i] - lo) >> shift) & mask], 1u);
        __syncthreads();
        const uint32_t first = scan_block<T / 64>(tid < 256 ? sh.boff[tid] : 0u, sh.w, &sum);
        if (tid < 256) sh.run[tid] = first;
        for (int64_t t0 = 0; t0 < m; t0 += STEP) {
            const int cnt = m - t0 < STEP ? (int)(m - t0) : STEP;
            for (int i = tid; i < T / 64 * 256; i += T) (&sh.wcnt[0][0])[i] = 0u;
            __syncthreads();
            uint32_t key[SLOW_ITEMS], val[SLOW_ITEMS], loc[SLOW_ITEMS];
            auto ok = [&](int j) { return w * (64 * SLOW_ITEMS) + j * 64 + lane < cnt; };
            auto dig = [&](int j) { return ((key[j] - lo) >> shift) & mask; };
#pragma unroll
            for (int j = 0; j < SLOW_ITEMS; j++) {
                const int i = w * (64 * SLOW_ITEMS) + j * 64 + lane;
                key[j] = ok(j) ? ks[t0 + i] : 0u;
                val[j] = ok(j) ? vs[t0 + i] : 0u;
            }
            rank_wave<SLOW_ITEMS, 8>(sh.wcnt[w], loc, dig, ok);
            __syncthreads();
            uint32_t tot = 0;
            if (tid < 256)
                for (int k = 0; k < T / 64; k++) {
                    const uint32_t c = sh.wcnt[k][tid];
                    sh.wcnt[k][tid] = tot;
                    tot += c;
                }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < SLOW_ITEMS; j++)
                if (ok(j)) {
                    const uint32_t dd = dig(j), g = sh.run[dd] + sh.wcnt[w][dd] + loc[j];
                    kd[g] = key[j];
                    vd[g] = val[j];
                }
            __syncthreads();
            if (tid < 256) sh.run[tid] += tot;
            __syncthreads();
        }
        uint32_t *t = ks;
        ks = kd;
        kd = t;
        t = vs;
        vs = vd;
        vd = t;
    }
    __syncthreads();
    for (int64_t i0 = 0; i0 < m; i0 += T) {
        const int64_t i = i0 + tid;
        const uint32_t v = i < m ? vs[i] : 0u, c = nt && i < m ? nt[v] : 0u;
        const uint32_t pre = scan_block<T / 64>(c, sh.w, &sum);
        if (i < m) {
            v0[start + i] = v;
            if (nt) {
                nt_sorted[start + i] = c;
                offsets[start + i] = base + pre;
            }
        }
        base += sum;
        __syncthreads();
    }
}

// A bucket of one depth is in order as it stands.  Its block and the blocks of the
// empty buckets before it (as many as splitters are equal to the depth, so parts are no
// larger than other buckets) write a part of it each: where a part's prefix starts
// follows from the tiles' sums.  b: the block's bucket, of one depth; start of vin, order,
// .. and base: those of the buckets from b on.
template <int T>
__device__ __attribute__((noinline)) void share_bucket(DsWs ws, int tiles, int b, const uint32_t *__restrict__ vin,
                                                       uint32_t *__restrict__ order, uint32_t base,
                                                       const uint32_t *__restrict__ nt, uint32_t *__restrict__ nt_sorted,
                                                       uint32_t *__restrict__ offsets, LocalShared<T> &sh) {
    static_assert(T >= NB && DS_LIGHT <= 256 * 2 * DT && DS_SMALL <= DT * 2 * DT && DEPTH_SORT_MAX <= DT * 4 * DT,
                  "a splitter and a tile for each thread");
    constexpr int I = 4;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // the run: its first splitter, and its bucket (the first splitter above the depth)
    const uint32_t depth = ws.split[b - 1], x = tid < NB - 1 ? ws.split[tid] : 0xFFFFFFFFu;
    const int first = __syncthreads_count(tid < NB - 1 && x < depth);
    const int own = __syncthreads_count(tid < NB - 1 && x <= depth);
    if (own == NB - 1 || ws.split[own] != depth + 1) return;   // (b is empty)
    const uint32_t m = ws.total[own], parts = (uint32_t)(own - first), k = (uint32_t)(b - 1 - first);
    if (m == 0) return;
    const uint32_t p0 = (uint32_t)((uint64_t)m * k / parts), p1 = (uint32_t)((uint64_t)m * (k + 1) / parts);
    uint32_t sum = 0, all;
    if (nt) {   // the tile counts before this part: whole tiles', then those of the tile it starts in
        const uint2 t = tid < tiles ? ws.part[tid * NB + own] : make_uint2(0u, 0u);
        const uint32_t at = scan_block<T / 64>(t.x, sh.w, &all);
        if (at + t.x <= p0) sum = t.y;
        else if (at <= p0) sh.boff[0] = at;
        __syncthreads();
        for (uint32_t i = sh.boff[0] + tid; i < p0; i += T) sum += nt[vin[i]];
        (void)scan_block<T / 64>(sum, sh.w, &all);
        base += all;
    }
    for (uint32_t i0 = p0; i0 < p1; i0 += I * T) {
        const uint32_t at = i0 + (uint32_t)(w * (64 * I) + lane);
        uint32_t val[I], cn[I];
#pragma unroll
        for (int j = 0; j < I; j++) val[j] = at + j * 64 < p1 ? vin[at + j * 64] : 0u;
#pragma unroll
        for (int j = 0; j < I; j++) cn[j] = nt && at + j * 64 < p1 ? nt[val[j]] : 0u;
        base = write_bucket<T, I>(val, cn, min(p1 - i0, (uint32_t)(I * T)), base, sh.w, order + i0,
                                  nt ? nt_sorted + i0 : nullptr, offsets + i0);
    }
}

// LDS of a bucket's sort: the cells', or the digit passes' and their reorder buffer.
template <int T, int ITEMS, int SB>
struct BucketShared {
    struct Digits {
        LocalShared<T> d;
        uint32_t buf[4 * T];
    };
    union {
        CellShared<T, T * ITEMS, SB> cells;
        Digits digits;
    };
};

// A bucket of m <= T * ITEMS keys in one block, by cells if they are even enough.
template <int T, int ITEMS, int MAXI, int SB, bool CULL = false>
__device__ __forceinline__ bool bucket_cells(const uint32_t *kin, const uint32_t *vin, uint32_t m, uint32_t base,
                                             const uint32_t *nt, uint32_t *order, uint32_t *nt_sorted,
                                             uint32_t *offsets, CellMap map, BucketShared<T, MAXI, SB> &sh) {
    return cell_sort<T, ITEMS, T * MAXI, SB, CULL>(kin, vin, m, base, nt, order, nt_sorted, offsets, map, sh.cells);
}

// One block per bucket: up to T * DS_ITEMS keys by cells, or where cells are too full by
// digit passes, of up to 4 T keys in LDS and of more in global memory; buckets of one
// depth as share_bucket says.
template <int T>
__global__ void __launch_bounds__(T, 4) k_ds_local(DsWs ws, int tiles, uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1,
                                                 const uint32_t *__restrict__ nt, uint32_t *__restrict__ nt_sorted,
                                                 uint32_t *__restrict__ offsets, uint32_t *__restrict__ n_keys) {
    constexpr int I = DS_ITEMS, SB = 4 * T;
    __shared__ BucketShared<T, I, SB> sh;
    __shared__ struct {
        uint32_t a[T / 64], b[T / 64], c[T / 64], m, kind;
    } pl;
    const int tid = threadIdx.x, b = (int)blockIdx.x;
    // this bucket's place: the totals and the tile-count sums before it; its own keys, and
    // whether they are of one depth (1) or the deepest (2)
    uint32_t first = 0, pre = 0, all = 0;
    if (tid < NB) {
        const uint32_t cn = ws.ntsum[tid], tot = ws.total[tid];
        const bool inner = tid > 0 && tid < NB - 1;
        const uint32_t lo = inner ? ws.split[tid - 1] : 0u, hi = inner ? ws.split[tid] : 0xFFFFFFFFu;
        if (tid == b) {
            pl.m = tot;
            pl.kind = hi - lo <= 1u ? 1u : hi == CULLED ? 2u : 0u;   // (as one_depth)
        }
        if (tid < b) {
            first += tot;
            pre += cn;
        }
        all = cn;
    }
    for (int o = 32; o > 0; o >>= 1) {
        first += (uint32_t)__shfl_xor((int)first, o, 64);
        pre += (uint32_t)__shfl_xor((int)pre, o, 64);
        all += (uint32_t)__shfl_xor((int)all, o, 64);
    }
    if ((tid & 63) == 0) {
        pl.a[tid >> 6] = first;
        pl.b[tid >> 6] = pre;
        pl.c[tid >> 6] = all;
    }
    __syncthreads();
    first = pre = all = 0;
    for (int k = 0; k < T / 64; k++) {
        first += pl.a[k];
        pre += pl.b[k];
        all += pl.c[k];
    }
    if (b == 0 && tid == 0 && nt) *n_keys = all;
    // (uniform: scalar bases for the bucket's addresses)
    const int64_t start = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)first);
    const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)pre);
    const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)pl.m);
    const uint32_t *kin = k1 + start, *vin = v1 + start;
    uint32_t *o = v0 + start, *ns = nt ? nt_sorted + start : nullptr, *off = offsets + start;
    const uint32_t kind = (uint32_t)__builtin_amdgcn_readfirstlane((int)pl.kind);
    if (kind == 1u) {
        share_bucket<T>(ws, tiles, b, vin, o, base, nt, ns, off, sh.digits.d);
        return;
    }
    if (m == 0) return;
    const CellMap map = b == 0 ? CELLS_FROM_HI : kind == 2u ? CELLS_FROM_LO : CELLS_EVEN;
    bool done = false;
    if (m <= T) done = bucket_cells<T, 1, I, SB>(kin, vin, m, base, nt, o, ns, off, map, sh);
    else if (m <= 4 * T) done = bucket_cells<T, 4, I, SB>(kin, vin, m, base, nt, o, ns, off, map, sh);
    else if (m <= 8 * T) done = bucket_cells<T, 8, I, SB>(kin, vin, m, base, nt, o, ns, off, map, sh);
    else if (m <= I * T) done = bucket_cells<T, I, I, SB>(kin, vin, m, base, nt, o, ns, off, map, sh);
    if (done) return;
    __syncthreads();
    if (m <= 4 * T) local_sort<T, 4>(kin, vin, m, base, nt, o, ns, off, sh.digits.d, sh.digits.buf);
    else slow_sort<T>(k0, v0, k1, v1, start, m, base, nt, nt_sorted, offsets, sh.digits.d);
}

// Up to DS_ONE entries in one block, straight from the depth keys.
__global__ void __launch_bounds__(DT) k_ds_one(const uint32_t *__restrict__ keys, uint32_t n,
                                               const uint32_t *__restrict__ nt, uint32_t *__restrict__ order,
                                               uint32_t *__restrict__ nt_sorted, uint32_t *__restrict__ offsets,
                                               uint32_t *__restrict__ n_keys) {
    constexpr int T = DT, SB = 4 * DT, I = (int)(DS_ONE / DT);
    __shared__ BucketShared<T, I, SB> sh;
    bool done;
    if (n <= T) done = bucket_cells<T, 1, I, SB, true>(keys, nullptr, n, 0u, nt, order, nt_sorted, offsets, CELLS_EVEN, sh);
    else if (n <= 2 * T) done = bucket_cells<T, 2, I, SB, true>(keys, nullptr, n, 0u, nt, order, nt_sorted, offsets, CELLS_EVEN, sh);
    else done = bucket_cells<T, I, I, SB, true>(keys, nullptr, n, 0u, nt, order, nt_sorted, offsets, CELLS_EVEN, sh);
    if (!done) {
        __syncthreads();
        local_sort<T, I, true>(keys, nullptr, n, 0u, nt, order, nt_sorted, offsets, sh.digits.d, sh.digits.buf);
    }
    __syncthreads();
    if (threadIdx.x == 0 && nt) *n_keys = offsets[n - 1] + nt_sorted[n - 1];   // the last entry's end
}

template <int R, int S, int T>
void ds_run(const uint32_t *keys, int64_t n, uint32_t *const dkeys[2], uint32_t *const dvals[2], const uint32_t *nt,
            uint32_t *nt_sorted, uint32_t *offsets, uint32_t *n_keys, void *wsp, hipStream_t s) {
    const int64_t tiles = (n + DT * R - 1) / (DT * R);
    const DsWs ws = ds_ws(wsp, tiles);
    const int rows = tiles <= DS_ROWS ? 1 : 0;
    const dim3 tg((unsigned)tiles), block(DT);
    hipLaunchKernelGGL((k_ds_up<R, S>), tg, block, 0, s, keys, n, ws, tiles, rows);
    if (!rows) hipLaunchKernelGGL(k_ds_scan, dim3(NB), dim3(256), 0, s, ws, tiles);
    hipLaunchKernelGGL((k_ds_down<R>), tg, block, 0, s, keys, nt, n, ws, tiles, rows, dkeys[1], dvals[1]);
    hipLaunchKernelGGL((k_ds_local<T>), dim3(NB), dim3(T), 0, s, ws, (int)tiles, dkeys[0], dvals[0], dkeys[1], dvals[1], nt, nt_sorted,
                       offsets, n_keys);
}

}  // namespace

size_t depth_sort_bytes(int64_t cap) {
    if (cap > DEPTH_SORT_MAX) cap = DEPTH_SORT_MAX;
    return (size_t)(3 * NB + (cap + 2 * DT - 1) / (2 * DT) * NB * 3) * 4;   // three words a bucket and tile of 2048 keys
}

int depth_sort(const uint32_t *depth_key, int64_t n, uint32_t *const dkeys[2], uint32_t *const dvals[2],
               const uint32_t *ntiles, uint32_t *nt_sorted, uint32_t *offsets, uint32_t *n_keys, void *ws,
               hipStream_t s) {
    if (n <= 0 || n > DEPTH_SORT_MAX) return -1;
    if (n <= DS_ONE)
        hipLaunchKernelGGL(k_ds_one, dim3(1), dim3(DT), 0, s, depth_key, (uint32_t)n, ntiles, dvals[0], nt_sorted, offsets,
                           n_keys);
    else if (n <= DS_LIGHT)
        ds_run<2, DT, 256>(depth_key, n, dkeys, dvals, ntiles, nt_sorted, offsets, n_keys, ws, s);
    else if (n <= DS_SMALL)
        ds_run<2, DT, DT>(depth_key, n, dkeys, dvals, ntiles, nt_sorted, offsets, n_keys, ws, s);
    else
        ds_run<4, 2 * DT, DT>(depth_key, n, dkeys, dvals, ntiles, nt_sorted, offsets, n_keys, ws, s);
    return 0;
}

AS_WARM_KERNEL(depth_sort)
