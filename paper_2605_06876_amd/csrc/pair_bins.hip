// Pairs of large renders, binned in two levels.
//
// A pair list sorted by bin moves every (bin, entry) pair through each of the
// sort's passes, although neighbouring bins hold mostly the same entries.
// Here the sort works on coarse bins of F x F bins (F 2 or 4), which hold two to
// four times fewer pairs; the pairs of the bins are written once, at the end:
//   sum     the pixel boxes gathered into depth order, and per 2048 ranks the
//           sums of the bins and of the coarse bins touched;
//   emit    every rank's coarse pairs: key = coarse bin id | the rectangle of
//           its bins that the entry touches, value = entry id;
//   sort    (radix.hip) stably on the coarse bin id: the rectangles ride along;
//   count   a block per coarse bin counts the pairs of each of its bins;
//   (scan)  the counts' exclusive prefix over the bins gives their list starts;
//   place   a block per coarse bin writes its bins' lists, in the order of
//           the coarse list, and the tiles' ranges.
// Stability carries over: a bin's list is the coarse list filtered, so keys,
// values, ranges and counts are those of the one-level sort bit for bit, also
// where the pair capacity cuts the render short (the cut is taken on the bins' pairs).
//
// Emission, sort and ranges against this (us, MI355X, with the gather of the
// tile counts into depth order where it is the sort's last pass): 82.8M pairs of
// eight views 1810 -> 700, 9.7M of one 1920x1080 view 175 -> 95.  What bounds
// it now: the placing, 208 us for 82.8M pairs (4.0 TB/s of a copy's 4.8), and the random read of the boxes
// (157 us for 8.2M entries).  Placing by a block per list in place of work items:
// 920 us, the lists are uneven; eight blocks per list 350 us.  Loading each
// round on its own: 1690 us, a wave's loads wait for the stores before them.
// Counting by ballots as the placing does: 67 us, by packed counts 28.  Emitting
// with lanes that search for the owner of their position: 105 us, by owner 89.
#include "internal.h"
#include "pair_count.h"

namespace {

constexpr int PB_THREADS = 256;
constexpr int PB_ROUNDS_SMALL = 2, PB_ROUNDS_BIG = 8;   // ranks per thread of sum and emit
constexpr int64_t PB_SMALL = 1 << 20;             // ranks up to which they take the fewer
constexpr int64_t PB_DIRECT = 2048;               // blocks up to which each sums the partials before it itself
constexpr uint32_t PB_OWN = 8;                    // coarse pairs that an entry's own lane writes
constexpr int PB_WAVES = 4;                       // waves of a block of count and place
constexpr int PB_BATCH = 6;                       // rounds of 64 pairs of a wave (place and count, 82.8M pairs / 0.6M: 236 / 12.5 us; 4: 246 / 11.7, 8: 238 / 13.4)
constexpr int PB_SLICE = 64 * PB_BATCH;
constexpr int PB_ITEM = PB_WAVES * PB_SLICE;      // pairs of a work item
// Items of a list are summed in groups as well, so that an item that looks up what
// the list holds before it reads a few sums however long the list is: 8M entries in two
// lists, counting and placing 168 us by items alone, 127 like this (spread over all lists 83);
// 8M in four lists around one point 197, 145.
constexpr uint32_t PB_GROUP = 64;
// Most blocks of count and of place, which loop over the items.  The placing's items
// are uneven and wait for their writes, so it takes many more blocks than
// are resident: 2048 blocks 245 us at 82.8M pairs, 16384 209.
constexpr int PB_GRID_COUNT = 2048, PB_GRID_PLACE = 16384;
constexpr int PB_LISTS = 63;                      // lists found by a block: a row of 16 lanes for each start, and the last one's end
constexpr uint32_t PB_ID = 0xFFFFFFu;             // key: coarse bin id in 24 bits, then x0, x1, y0, y1 of two bits

// Bins and coarse bins touched by an entry, from its box (x0 > x1 when culled).
struct BinRect {
    int fx0, fx1, fy0, fy1;
};
__device__ __forceinline__ BinRect bin_rect(uint32_t lo, uint32_t hi, int bs) {
    // (arithmetic shifts: the empty box ends at -1)
    return BinRect{(int16_t)(lo & 0xFFFFu) >> bs, (int16_t)(hi & 0xFFFFu) >> bs, (int16_t)(lo >> 16) >> bs,
                   (int16_t)(hi >> 16) >> bs};
}
// (bins << 32) | coarse bins: both counts in one sum (pair_count.h)
__device__ __forceinline__ uint64_t rect_counts(const BinRect &b, int cs) {
    const uint32_t f = (uint32_t)((b.fx1 - b.fx0 + 1) * (b.fy1 - b.fy0 + 1));
    const uint32_t c = f ? (uint32_t)(((b.fx1 >> cs) - (b.fx0 >> cs) + 1) * ((b.fy1 >> cs) - (b.fy0 >> cs) + 1)) : 0u;
    return ((uint64_t)f << 32) | c;
}

// Prefix and sum over the wave of the counts of up to 8 entries a lane, the
// halves apart and exact: an entry touches at most 2^22 bins (a view is at most
// 32,767 pixels a side), 512 of them 2^31.  Sums beyond a wave saturate.
__device__ __forceinline__ uint64_t wave_prefix2(uint64_t v) {
    return ((uint64_t)wave_prefix((uint32_t)(v >> 32)) << 32) | wave_prefix((uint32_t)v);
}
__device__ __forceinline__ uint64_t last_lane2(uint64_t v) {
    return ((uint64_t)last_lane((uint32_t)(v >> 32)) << 32) | last_lane((uint32_t)v);
}
__device__ __forceinline__ uint64_t wave_sum(uint64_t v) { return last_lane2(wave_prefix2(v)); }
// The same of saturated sums: the bins in two parts of 16 bits, whose sums do not carry.
__device__ __forceinline__ uint64_t wave_sum_sat(uint64_t v) {
    const uint32_t b = (uint32_t)(v >> 32);
    const uint64_t bins = ((uint64_t)last_lane(wave_prefix(b >> 16)) << 16) + last_lane(wave_prefix(b & 0xFFFFu));
    return bins >> 32 ? ~0ull : (bins << 32) | last_lane(wave_prefix((uint32_t)v));
}
// Counts added: with SAT saturating, else of a render whose entries could touch all bins
// of their views without the sum reaching 2^32 (1M entries, 1040 bins: 10.3 us, 11.0 saturating).
template <bool SAT>
__device__ __forceinline__ uint64_t add(uint64_t a, uint64_t b) {
    return SAT ? sat_add(a, b) : a + b;
}
// The waves' sums added (every thread gets it); s of PB_THREADS / 64 words.
template <bool SAT>
__device__ __forceinline__ uint64_t block_sum(uint64_t wave, uint64_t *s) {
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = wave;
    __syncthreads();
    uint64_t t = 0;
    for (int k = 0; k < PB_THREADS / 64; k++) t = add<SAT>(t, s[k]);
    __syncthreads();
    return t;
}

// Exclusive prefix of the blocks' sums, in place, by one block.
__global__ void __launch_bounds__(PB_THREADS) k_pairs_scan(uint64_t *__restrict__ partials, int64_t nb) {
    constexpr int ITEMS = 8, W = PB_THREADS / 64;
    __shared__ uint64_t s_w[2][W];   // (one barrier a turn: the next writes the other half)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t carry = 0;
    int flip = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += PB_THREADS * ITEMS, flip ^= 1) {
        const int64_t base = c0 + (int64_t)threadIdx.x * ITEMS;
        uint64_t v[ITEMS], sum = 0;
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            v[k] = base + k < nb ? partials[base + k] : 0ull;
            sum = sat_add(sum, v[k]);
        }
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t t = __shfl_up(sum, o, 64);
            if (lane >= o) sum = sat_add(sum, t);
        }
        if (lane == 63) s_w[flip][w] = sum;
        const uint64_t up = __shfl_up(sum, 1, 64);
        __syncthreads();
        uint64_t run = carry;
        for (int k = 0; k < W; k++) {
            const uint64_t x = s_w[flip][k];
            if (k < w) run = sat_add(run, x);
            carry = sat_add(carry, x);
        }
        if (lane > 0) run = sat_add(run, up);
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            if (base + k < nb) partials[base + k] = run;
            run = sat_add(run, v[k]);
        }
    }
}

// The one random read of the path: a box per rank, kept in depth order for the emission.
template <int R>
__global__ void __launch_bounds__(PB_THREADS) k_pairs_sum(int64_t n, const uint32_t *__restrict__ order, int bs, int cs,
                                                          const uint2 *__restrict__ box, uint32_t *__restrict__ box_lo,
                                                          uint32_t *__restrict__ box_hi, uint64_t *__restrict__ partials,
                                                          uint32_t *__restrict__ n_items) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_items = 0u;   // for k_bins_lists
    __shared__ uint64_t s_w[PB_THREADS / 64];
    const int64_t base = (int64_t)blockIdx.x * (PB_THREADS * R) + threadIdx.x;
    uint32_t e[R];
    uint2 b[R];
#pragma unroll
    for (int j = 0; j < R; j++) e[j] = base + j * PB_THREADS < n ? order[base + j * PB_THREADS] : 0u;
#pragma unroll
    for (int j = 0; j < R; j++) b[j] = box[e[j]];   // (ranks past the end read entry 0)
    uint64_t sum = 0;
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int64_t r = base + j * PB_THREADS;
        if (r < n) {
            box_lo[r] = b[j].x;
            box_hi[r] = b[j].y;
            sum += rect_counts(bin_rect(b[j].x, b[j].y, bs), cs);
        }
    }
    sum = block_sum<true>(wave_sum(sum), s_w);
    if (threadIdx.x == 0) partials[blockIdx.x] = sum;
}

// Coarse pairs in depth order: consecutive ranks own consecutive positions.
// Most entries touch one to four coarse bins, so each lane writes the first
// PB_OWN pairs of its own rank (a wave's stores of one step lie within a few
// lines), and the wave together what a larger entry has beyond them.
template <int R, bool SAT>
__global__ void __launch_bounds__(PB_THREADS) k_pairs_emit(int64_t n, const uint32_t *__restrict__ order,
                                                           const ViewTable vt, const CoarseBins cb,
                                                           const uint32_t *__restrict__ box_lo,
                                                           const uint32_t *__restrict__ box_hi,
                                                           const uint64_t *__restrict__ partials, int scanned,
                                                           int64_t key_cap, uint32_t *__restrict__ keys,
                                                           uint32_t *__restrict__ vals, uint32_t *__restrict__ n_keys,
                                                           const PairReport report) {
    constexpr int W = PB_THREADS / 64;
    __shared__ uint64_t s_w[W];
    __shared__ int s_base[AS_MAX_VIEWS], s_pitch[AS_MAX_VIEWS];   // of the lanes' views (read by lane: not from the arguments)
    if (threadIdx.x < AS_MAX_VIEWS) {
        s_base[threadIdx.x] = cb.base[threadIdx.x];
        s_pitch[threadIdx.x] = cb.x[threadIdx.x];
    }
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int bs = vt.bin_shift, cs = cb.shift;
    const int64_t r0 = (int64_t)blockIdx.x * (PB_THREADS * R) + w * (R * 64) + lane;
    uint32_t lo[R], hi[R], id[R];
    uint64_t sum = 0;
#pragma unroll
    for (int j = 0; j < R; j++) {
        const int64_t r = r0 + j * 64;
        lo[j] = r < n ? box_lo[r] : 0u;
        hi[j] = r < n ? box_hi[r] : 0xFFFFFFFFu;   // the empty box
        id[j] = r < n ? order[r] : 0u;
    }
#pragma unroll
    for (int j = 0; j < R; j++) sum += rect_counts(bin_rect(lo[j], hi[j], bs), cs);
    // (bins << 32 | coarse bins) before this block, then before this wave
    uint64_t pre = 0;
    if (scanned) {
        pre = partials[blockIdx.x];
    } else {
        for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += PB_THREADS) pre = add<SAT>(pre, partials[b]);
        pre = block_sum<SAT>(SAT ? wave_sum_sat(pre) : wave_sum(pre), s_w);
    }
    sum = wave_sum(sum);
    if (lane == 0) s_w[w] = sum;
    __syncthreads();
    uint64_t all = pre;
    for (int k = 0; k < W; k++) {
        const uint64_t x = s_w[k];
        if (k < w) pre = add<SAT>(pre, x);
        all = add<SAT>(all, x);
    }
    // n_keys: the pairs of the bins needed and written, and the coarse pairs written
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        n_keys[0] = (uint32_t)(all >> 32);
        send_report(report, (uint32_t)(all >> 32));
        if ((all >> 32) <= (uint64_t)key_cap) {
            n_keys[1] = (uint32_t)(all >> 32);
            n_keys[2] = (uint32_t)all;
        }
    }
    const int m = (1 << cs) - 1;
#pragma unroll
    for (int j = 0; j < R; j++) {
        const BinRect b = bin_rect(lo[j], hi[j], bs);
        const uint64_t c = rect_counts(b, cs), inc = wave_prefix2(c), at = add<SAT>(pre, inc - c);
        pre = add<SAT>(pre, last_lane2(inc));
        const PairCut cut = pair_cut(at, c, (uint64_t)key_cap);
        if (cut.crosses) {
            n_keys[1] = (uint32_t)(at >> 32);
            n_keys[2] = (uint32_t)at;
        }
        const uint32_t ct = cut.kept ? (uint32_t)c : 0u, coff = (uint32_t)at;
        if (!__builtin_amdgcn_ballot_w64(ct != 0)) continue;
        const int v = view_of_entry(vt, id[j]), pitch = s_pitch[v], base = s_base[v];
        const int cx0 = b.fx0 >> cs, cx1 = b.fx1 >> cs, cy0 = b.fy0 >> cs;
        // pair (cx, cy) of an entry: the coarse bin and the entry's bins inside it
        auto key_of = [&](int bin0, int p, int cx, int cy, int fx0, int fx1, int fy0, int fy1) {
            const int x0 = max(fx0 - (cx << cs), 0), x1 = min(fx1 - (cx << cs), m);
            const int y0 = max(fy0 - (cy << cs), 0), y1 = min(fy1 - (cy << cs), m);
            return (uint32_t)(bin0 + cy * p + cx) | ((uint32_t)(x0 | (x1 << 2) | (y0 << 4) | (y1 << 6)) << 24);
        };
        int cx = cx0, cy = cy0;
        for (uint32_t t = 0; t < PB_OWN && __builtin_amdgcn_ballot_w64(t < ct); t++) {
            if (t < ct) {
                keys[coff + t] = key_of(base, pitch, cx, cy, b.fx0, b.fx1, b.fy0, b.fy1);
                vals[coff + t] = id[j];
            }
            const bool wrap = cx == cx1;
            cx = wrap ? cx0 : cx + 1;
            cy += wrap ? 1 : 0;
        }
        for (uint64_t big = __builtin_amdgcn_ballot_w64(ct > PB_OWN); big; big &= big - 1) {
            const int l = __builtin_ctzll(big);
            auto get = [&](int x) { return __builtin_amdgcn_readlane(x, l); };
            const uint32_t lct = (uint32_t)get((int)ct), loff = (uint32_t)get((int)coff), lid = (uint32_t)get((int)id[j]);
            const int fx0 = get(b.fx0), fx1 = get(b.fx1), fy0 = get(b.fy0), fy1 = get(b.fy1);
            const int bin0 = get(base), p = get(pitch);
            const uint32_t cw = (uint32_t)((fx1 >> cs) - (fx0 >> cs) + 1);
            for (uint32_t q = PB_OWN + lane; q < lct; q += 64) {
                const uint32_t qy = q / cw;
                keys[loff + q] = key_of(bin0, p, (fx0 >> cs) + (int)(q - qy * cw), (fy0 >> cs) + (int)qy, fx0, fx1, fy0, fy1);
                vals[loff + q] = lid;
            }
        }
    }
}

// Bit dy * F + dx for every bin (dx, dy) of the key's rectangle.
template <int F>
__device__ __forceinline__ uint32_t rect_mask(uint32_t key) {
    const uint32_t x0 = (key >> 24) & 3u, x1 = (key >> 26) & 3u, y0 = (key >> 28) & 3u, y1 = key >> 30;
    const uint32_t row = (2u << x1) - (1u << x0);
    // the rows y0 .. y1 as one bit every F bits, from y0 F on
    const uint32_t ones = F == 4 ? 0x1111u : 0x5u;
    const uint32_t rows = (ones << (F * y0)) & ((2u << (F * y1)) - 1u);
    return row * rows;
}

// First of the n keys whose coarse bin is not below `bin`: each row of 16 lanes
// searches for its own bin, splitting the range 16 ways a step (n <= 2^32 in
// eight steps; 64 ways would read three times the lines, 27 us against 12 for 4,080 lists).
__device__ __forceinline__ uint32_t coarse_bound(const uint32_t *__restrict__ keys, uint32_t n, uint32_t bin) {
    const uint32_t lane = threadIdx.x & 63, sub = lane & 15;
    uint32_t lo = 0, hi = n;
    while (__builtin_amdgcn_ballot_w64(lo < hi)) {
        const uint32_t step = (uint32_t)(((uint64_t)(hi - lo) + 15) / 16);
        const uint64_t p = (uint64_t)lo + (uint64_t)(sub + 1) * step - 1;
        const bool below = lo < hi && p < hi && (keys[p] & PB_ID) < bin;
        const uint64_t all = __builtin_amdgcn_ballot_w64(below);
        const uint32_t cnt = (uint32_t)__popc((uint32_t)(all >> (lane & 48)) & 0xFFFFu);
        if (lo < hi) {
            const uint64_t top = (uint64_t)lo + (uint64_t)(cnt + 1) * step - 1;
            const uint64_t bot = (uint64_t)lo + (uint64_t)cnt * step;
            lo = bot < hi ? (uint32_t)bot : hi;
            hi = top < hi ? (uint32_t)top : hi;
        }
    }
    return lo;
}

// Coarse bin `cid`: its view, and its bin (0, 0) with the number of its bins
// that lie in the view.
struct CoarsePlace {
    int bin0, pitch, w, h;
};
__device__ __forceinline__ CoarsePlace coarse_place(const ViewTable &vt, const CoarseBins &cb, int cid) {
    int v = 0;
    for (int k = 1; k < vt.n_views; k++) v += cid >= cb.base[k] ? 1 : 0;
    const int l = cid - cb.base[v], cy = l / cb.x[v], cx = l - cy * cb.x[v];
    const int bx = vt.bins_x[v], by = (vt.bin_base[v + 1] - vt.bin_base[v]) / bx;
    return CoarsePlace{vt.bin_base[v] + (cy << cb.shift) * bx + (cx << cb.shift), bx, bx - (cx << cb.shift),
                       by - (cy << cb.shift)};
}

// The coarse lists, cut into work items of PB_ITEM pairs: a row of lanes finds
// each list's start, and each list takes its items' places from a counter (which
// list gets which is left to chance, and shows in nothing).  An item is
// (coarse bin, part of its list, list start, list length).  Also clears the
// bins' counts and the groups' for the launch that adds them, and the tiles' ranges.
__global__ void __launch_bounds__(1024) k_bins_lists(const uint32_t *__restrict__ keys,
                                                     const uint32_t *__restrict__ n_keys, int64_t key_cap, int cbins,
                                                     uint4 *__restrict__ items, uint32_t *__restrict__ n_items,
                                                     uint32_t *__restrict__ counts, int64_t bins,
                                                     uint32_t *__restrict__ groups, int64_t group_words,
                                                     uint32_t *__restrict__ ranges, int64_t range_words) {
    __shared__ uint32_t s_at[PB_LISTS + 1], s_item[PB_LISTS + 1];
    const int64_t t0 = (int64_t)blockIdx.x * 1024 + threadIdx.x, tn = (int64_t)gridDim.x * 1024;
    for (int64_t i = t0; i < bins; i += tn) counts[i] = 0u;
    for (int64_t i = t0; i < group_words; i += tn) groups[i] = 0u;
    for (int64_t i = t0; i < range_words; i += tn) ranges[i] = 0u;
    const int w = (int)(threadIdx.x >> 4), sub = (int)(threadIdx.x & 15);
    const int cid = (int)blockIdx.x * PB_LISTS + w;
    const uint32_t p = coarse_bound(keys, (uint32_t)min((int64_t)n_keys[2], key_cap), (uint32_t)cid);   // (bins past the last end where it ends)
    if (sub == 0) s_at[w] = p;
    __syncthreads();
    if (w == PB_LISTS || cid >= cbins) return;
    const uint32_t m = s_at[w + 1] - p, ni = (m + PB_ITEM - 1) / PB_ITEM;
    if (ni == 0) return;
    if (sub == 0) s_item[w] = atomicAdd(n_items, ni);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t at = s_item[w];
    for (uint32_t k = sub; k < ni; k += 16) items[at + k] = make_uint4((uint32_t)cid, k, p, m);
}

// The first group of the list whose first item is `first`: groups of lists after one
// another do not overlap (rounding up a first item and down a number of items).
__device__ __forceinline__ uint32_t first_group(uint32_t first) { return (first + PB_GROUP - 1) / PB_GROUP; }

// Pairs of each bin in every wave's slice of an item, in the item and in its group,
// and the bins' sums.
template <int F>
__global__ void __launch_bounds__(PB_WAVES * 64) k_bins_count(const uint32_t *__restrict__ keys, const ViewTable vt,
                                                              const CoarseBins cb, const uint4 *__restrict__ items,
                                                              const uint32_t *__restrict__ n_items,
                                                              uint32_t *__restrict__ slices, uint32_t *__restrict__ sums,
                                                              uint32_t *__restrict__ groups, uint32_t *__restrict__ counts) {
    constexpr int NC = F * F;
    __shared__ uint32_t s_c[2][PB_WAVES][4][4];   // per wave and row of 16 lanes: 16 counts of a byte
    static_assert(PB_BATCH * 16 < 256 && PB_BATCH < 16, "counts of a lane in four bits, of a row in eight");
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t ni = *n_items;
    int flip = 0;
    for (uint32_t it = blockIdx.x; it < ni; it += gridDim.x, flip ^= 1) {
        const uint4 item = items[it];
        const uint32_t m = item.w, i0 = min(m, item.y * PB_ITEM + (uint32_t)w * PB_SLICE), i1 = min(m, i0 + PB_SLICE);
        uint32_t key[PB_BATCH], top = 0, bot = 0;   // rows 0, 1 and 2, 3 of 4 x 4 counts of four bits
#pragma unroll
        for (int j = 0; j < PB_BATCH; j++) key[j] = keys[item.z + min(i0 + j * 64 + lane, m - 1)];
#pragma unroll
        for (int j = 0; j < PB_BATCH; j++) {
            const uint32_t k = key[j], x0 = (k >> 24) & 3u, x1 = (k >> 26) & 3u, y0 = (k >> 28) & 3u, y1 = k >> 30;
            uint32_t row = (0x1111u << (4 * x0)) & (0xFFFFu >> (12 - 4 * x1));
            row = i0 + j * 64 + lane < i1 ? row : 0u;
            const uint32_t rows = (2u << y1) - (1u << y0);
            top += __umul24(row, (rows & 1u) | ((rows & 2u) << 15));
            if (F == 4) bot += __umul24(row, ((rows >> 2) & 1u) | ((rows & 8u) << 13));
        }
        // the wave's sums by row of lanes: even and odd columns in bytes
        const uint32_t q[4] = {row_prefix(top & 0x0F0F0F0Fu), row_prefix((top >> 4) & 0x0F0F0F0Fu),
                               F == 4 ? row_prefix(bot & 0x0F0F0F0Fu) : 0u,
                               F == 4 ? row_prefix((bot >> 4) & 0x0F0F0F0Fu) : 0u};
        if ((lane & 15) == 15)
#pragma unroll
            for (int k = 0; k < 4; k++) s_c[flip][w][lane >> 4][k] = q[k];
        __syncthreads();   // (one a turn: the next writes the other half)
        if (tid < PB_WAVES * NC) {
            const int sw = tid / NC, k = tid % NC, c = (k / F) * 4 + k % F;   // wave, bin, its place in the 4 x 4
            uint32_t t = 0;
#pragma unroll
            for (int r = 0; r < 4; r++) t += (s_c[flip][sw][r][2 * (c / 8) + c % 2] >> (8 * (c / 2 % 4))) & 0xFFu;
            slices[((size_t)it * PB_WAVES + sw) * NC + k] = t;
            for (int o = NC; o < PB_WAVES * NC; o *= 2) t += (uint32_t)__shfl_xor((int)t, o, 64);
            if (sw == 0) {
                sums[(size_t)it * NC + k] = t;
                // (the groups that are whole; the items of a list's last few are read one by one)
                const uint32_t g = item.y / PB_GROUP;
                if (t && g < m / (PB_GROUP * PB_ITEM)) atomicAdd(groups + (size_t)(first_group(it - item.y) + g) * NC + k, t);
                const CoarsePlace p = coarse_place(vt, cb, (int)item.x);
                if (t) atomicAdd(counts + p.bin0 + (k / F) * p.pitch + k % F, t);   // (bins past the border hold no pair)
            }
        }
    }
}

// Each wave walks its slice of an item and appends every pair to the lists of
// the bins in its rectangle: a ballot per bin gives the places of a round's
// pairs, the wave's place in each list is a scalar.
template <int F>
__global__ void __launch_bounds__(PB_WAVES * 64) k_bins_place(const uint32_t *__restrict__ ckeys,
                                                              const uint32_t *__restrict__ cvals, const ViewTable vt,
                                                              const CoarseBins cb, const uint4 *__restrict__ items,
                                                              const uint32_t *__restrict__ n_items,
                                                              const uint32_t *__restrict__ slices,
                                                              const uint32_t *__restrict__ sums,
                                                              const uint32_t *__restrict__ groups,
                                                              const uint32_t *__restrict__ starts,
                                                              const uint32_t *__restrict__ counts,
                                                              uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                              uint32_t *__restrict__ ranges) {
    constexpr int NC = F * F, G = PB_WAVES * 64 / NC;
    __shared__ uint32_t s_sum[G][NC], s_from[PB_WAVES + 1][NC];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t ni = *n_items;
    for (uint32_t it = blockIdx.x; it < ni; it += gridDim.x) {
        const uint4 item = items[it];
        const uint32_t part = item.y, m = item.w;
        const uint32_t i0 = min(m, part * PB_ITEM + (uint32_t)w * PB_SLICE), i1 = min(m, i0 + PB_SLICE);
        // Stores and loads of a wave return in order: all loads come before the stores.
        uint32_t key[PB_BATCH], val[PB_BATCH];
#pragma unroll
        for (int j = 0; j < PB_BATCH; j++) {
            const uint32_t at = item.z + min(i0 + j * 64 + lane, m - 1);
            key[j] = ckeys[at];
            val[j] = cvals[at];
        }
        const CoarsePlace p = coarse_place(vt, cb, (int)item.x);
        // the pairs of each bin in the list's items before this one
        uint32_t pre = 0;
        const uint32_t first = it - part, gs = part / PB_GROUP;
        for (uint32_t k = (uint32_t)(tid / NC); k < gs; k += G) pre += groups[(size_t)(first_group(first) + k) * NC + tid % NC];
        for (uint32_t k = gs * PB_GROUP + (uint32_t)(tid / NC); k < part; k += G) pre += sums[(size_t)(first + k) * NC + tid % NC];
        s_sum[tid / NC][tid % NC] = pre;
        uint32_t own[PB_WAVES], s0 = 0, all = 0;
        const int dx = tid % F, dy = tid / F, bin = p.bin0 + dy * p.pitch + dx;
        const bool mine = tid < NC && dx < p.w && dy < p.h;
        if (tid < NC) {
#pragma unroll
            for (int k = 0; k < PB_WAVES; k++) own[k] = slices[((size_t)it * PB_WAVES + k) * NC + tid];
            if (mine) {
                s0 = starts[bin];
                if (part == 0) all = counts[bin];
            }
        }
        __syncthreads();
        if (tid < NC) {
            uint32_t at = s0;
#pragma unroll
            for (int k = 0; k < G; k++) at += s_sum[k][tid];
#pragma unroll
            for (int k = 0; k < PB_WAVES; k++) {
                s_from[k][tid] = at;
                at += own[k];
            }
            s_from[PB_WAVES][tid] = at;
            if (all) {
                set_bin_range(vt, (uint32_t)bin, 0, s0, ranges);
                set_bin_range(vt, (uint32_t)bin, 1, s0 + all, ranges);
            }
        }
        __syncthreads();
        uint32_t at[NC];
#pragma unroll
        for (int k = 0; k < NC; k++) at[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_from[w][k]);
#pragma unroll
        for (int j = 0; j < PB_BATCH; j++) {
            if (i0 + j * 64 >= i1) break;   // wave-uniform
            const uint32_t mask = i0 + j * 64 + lane < i1 ? rect_mask<F>(key[j]) : 0u;
#pragma unroll
            for (int k = 0; k < NC; k++) {
                const bool on = (mask >> k) & 1u;
                const uint64_t b = __ballot(on);
                if (on) {
                    const uint32_t before =
                        __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                    (vals + at[k])[before] = val[j];
                }
                at[k] += (uint32_t)__popcll(b);
            }
        }
        // the item's keys, one value per bin
#pragma unroll
        for (int k = w; k < NC; k += PB_WAVES) {
            const uint32_t id = (uint32_t)(p.bin0 + (k / F) * p.pitch + k % F), end = s_from[PB_WAVES][k];
            for (uint32_t i = s_from[0][k] + lane; i < end; i += 64) keys[i] = id;
        }
        __syncthreads();   // the next turn writes s_sum and s_from
    }
}

// The scratch: the items (at most one per coarse bin and one per PB_ITEM pairs),
// the pairs of each bin by slice, by item and by group, the bins' counts and starts,
// and the number of items.
struct PbWs {
    uint4 *items;
    uint32_t *slices, *sums, *groups, *counts, *starts, *n_items;
};
int64_t most_groups(int64_t items) { return items / PB_GROUP + 1; }
int64_t most_items(int64_t cbins, int64_t key_cap) { return cbins + key_cap / PB_ITEM; }
PbWs pb_ws(void *ws, const CoarseBins &cb, int64_t key_cap, int64_t bins) {
    const int64_t ni = most_items(cb.bins, key_cap), nc = (int64_t)1 << (2 * cb.shift);
    uint4 *items = reinterpret_cast<uint4 *>(ws);
    uint32_t *p = reinterpret_cast<uint32_t *>(items + ni);
    uint32_t *sums = p + ni * PB_WAVES * nc, *groups = sums + ni * nc, *counts = groups + most_groups(ni) * nc;
    return PbWs{items, p, sums, groups, counts, counts + bins, counts + 2 * bins};
}

int64_t fill_coarse(const ViewTable &vt, int shift, CoarseBins *cb) {
    const int f = 1 << shift;
    int64_t bins = 0;
    cb->shift = shift;
    for (int v = 0; v < vt.n_views; v++) {
        const int bx = vt.bins_x[v], by = (vt.bin_base[v + 1] - vt.bin_base[v]) / bx;
        cb->base[v] = (int32_t)bins;
        cb->x[v] = (bx + f - 1) / f;
        bins += (int64_t)cb->x[v] * ((by + f - 1) / f);
    }
    cb->bins = (int32_t)bins;
    return bins;
}

template <int R>
void pairs_emit(int64_t n, const uint32_t *order, const ViewTable &vt, const CoarseBins &cb, const int16_t *box,
                uint32_t *box_lo, uint32_t *box_hi, int64_t key_cap, uint32_t *keys, uint32_t *vals, uint32_t *n_keys,
                const PairReport &report, uint64_t *partials, uint32_t *n_items, hipStream_t s) {
    const int64_t nb = (n + PB_THREADS * R - 1) / (PB_THREADS * R);
    const dim3 grid((unsigned)nb), block(PB_THREADS);
    hipLaunchKernelGGL((k_pairs_sum<R>), grid, block, 0, s, n, order, vt.bin_shift, cb.shift,
                       reinterpret_cast<const uint2 *>(box), box_lo, box_hi, partials, n_items);
    const int scanned = nb > PB_DIRECT;
    if (scanned) hipLaunchKernelGGL(k_pairs_scan, dim3(1), block, 0, s, partials, nb);
    int64_t most = 0;   // bins of a view
    for (int v = 0; v < vt.n_views; v++) most = most > vt.bin_base[v + 1] - vt.bin_base[v] ? most : vt.bin_base[v + 1] - vt.bin_base[v];
    if (n * most <= MAX_PAIR_CAP)
        hipLaunchKernelGGL((k_pairs_emit<R, false>), grid, block, 0, s, n, order, vt, cb, box_lo, box_hi, partials, scanned,
                           key_cap, keys, vals, n_keys, report);
    else
        hipLaunchKernelGGL((k_pairs_emit<R, true>), grid, block, 0, s, n, order, vt, cb, box_lo, box_hi, partials, scanned,
                           key_cap, keys, vals, n_keys, report);
}

}  // namespace

size_t pairs_tmp_bytes(int64_t n) {
    const int64_t small = n < PB_SMALL ? n : PB_SMALL;
    const int64_t a = small / (PB_THREADS * PB_ROUNDS_SMALL) + 1, b = n / (PB_THREADS * PB_ROUNDS_BIG) + 1;
    return (size_t)(a > b ? a : b) * 8 + 256;
}

size_t coarse_bins_bytes(int64_t tiles, int64_t key_cap) {
    // Bins are at most the tiles, and coarse_bins() takes at most two bins'
    // worth of slots per bin; per item and slot PB_WAVES + 1 words, and one per group.
    static_assert(16 <= PB_GROUP, "at most a word of the groups per item");
    const int64_t per_item = 4 + (PB_WAVES + 1) * 16 + 1;
    return (size_t)(tiles * (4 + 2 * (PB_WAVES + 1) + 1 + 2) + key_cap / PB_ITEM * per_item + 16 + 1) * 4 + 256;
}

// Two launches more than the one-level path, against the pairs' traffic
// (render of one view, us, two levels / one, by pairs): 0.6M 159 / 150, 1.0M
// 181 / 177, 1.7M 208 / 210, 2.7M 246 / 258, 4.7M 350 / 383, 7.0M 398 / 448,
// 14.1M 937 / 1071, 21.2M 1056 / 1290.  The host knows the pairs by the frame's
// capacity, which is a few times what a render needs; few entries leave the
// emission's blocks too few.
//
// Coarse bins of 4 x 4 bins, or of 2 x 2 where that leaves fewer than 256 of
// them: fewer lists are too few places at once for a sort pass's writes (130
// lists of a 400x300 view, 1.3M pairs: 229 / 215).  Skinny or tiny views,
// where the coarse grid is mostly border, stay with one level.
bool coarse_bins(const ViewTable &vt, int64_t n, int64_t key_cap, CoarseBins *cb) {
    if (n < PAIR_BINS_ENTRIES || key_cap < PAIR_BINS_PAIRS || key_cap > MAX_PAIR_CAP) return false;
    const int64_t bins = vt.bin_base[vt.n_views];
    int64_t c = fill_coarse(vt, 2, cb);
    if (c < PAIR_BINS_LISTS) c = fill_coarse(vt, 1, cb);
    return c >= PAIR_BINS_LISTS && c <= (int64_t)PB_ID && (c << (2 * cb->shift)) <= 2 * bins;
}

void launch_pairs_emit(int64_t n, const uint32_t *order, const ViewTable &vt, const CoarseBins &cb, const int16_t *box,
                       uint32_t *box_lo, uint32_t *box_hi, int64_t key_cap, uint32_t *keys, uint32_t *vals,
                       uint32_t *n_keys, const PairReport &report, void *ws, void *tmp, hipStream_t s) {
    uint32_t *n_items = pb_ws(ws, cb, key_cap, vt.bin_base[vt.n_views]).n_items;
    uint64_t *partials = reinterpret_cast<uint64_t *>(tmp);
    if (n <= PB_SMALL)
        pairs_emit<PB_ROUNDS_SMALL>(n, order, vt, cb, box, box_lo, box_hi, key_cap, keys, vals, n_keys, report, partials,
                                    n_items, s);
    else
        pairs_emit<PB_ROUNDS_BIG>(n, order, vt, cb, box, box_lo, box_hi, key_cap, keys, vals, n_keys, report, partials,
                                    n_items, s);
}

void launch_bins_place(const ViewTable &vt, const CoarseBins &cb, int64_t key_cap, const uint32_t *ckeys,
                       const uint32_t *cvals, uint32_t *keys, uint32_t *vals, const uint32_t *n_keys, uint32_t *ranges,
                       int64_t n_tiles, void *ws, void *tmp, hipStream_t s) {
    const int64_t bins = vt.bin_base[vt.n_views], most = most_items(cb.bins, key_cap);
    const PbWs p = pb_ws(ws, cb, key_cap, bins);
    const dim3 grid((unsigned)(most < PB_GRID_COUNT ? most : PB_GRID_COUNT)), block(PB_WAVES * 64);
    const dim3 wide((unsigned)(most < PB_GRID_PLACE ? most : PB_GRID_PLACE));
    hipLaunchKernelGGL(k_bins_lists, dim3((unsigned)(cb.bins + PB_LISTS - 1) / PB_LISTS), dim3(1024), 0, s, ckeys, n_keys,
                       key_cap, cb.bins, p.items, p.n_items, p.counts, bins, p.groups,
                       most_groups(most) << (2 * cb.shift), ranges, 2 * n_tiles);
    if (cb.shift == 2)
        hipLaunchKernelGGL(k_bins_count<4>, grid, block, 0, s, ckeys, vt, cb, p.items, p.n_items, p.slices, p.sums, p.groups,
                           p.counts);
    else
        hipLaunchKernelGGL(k_bins_count<2>, grid, block, 0, s, ckeys, vt, cb, p.items, p.n_items, p.slices, p.sums, p.groups,
                           p.counts);
    scan_u32(p.counts, p.starts, bins, nullptr, tmp, s);
    if (cb.shift == 2)
        hipLaunchKernelGGL(k_bins_place<4>, wide, block, 0, s, ckeys, cvals, vt, cb, p.items, p.n_items, p.slices, p.sums,
                           p.groups, p.starts, p.counts, keys, vals, ranges);
    else
        hipLaunchKernelGGL(k_bins_place<2>, wide, block, 0, s, ckeys, cvals, vt, cb, p.items, p.n_items, p.slices, p.sums,
                           p.groups, p.starts, p.counts, keys, vals, ranges);
}

AS_WARM_KERNEL(pair_bins)
