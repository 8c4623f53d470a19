// Error region partitioning of one sampled view (Sec. 4.1): normalised L1 error
// (Eq. (l1map)), metric map, attribution counts, erosion, error bands, 8-connected
// regions of equal (dominant candidate, band) (Eq. (error-region)), the area
// filter (Eq. (min_region_area)) and the region statistics.
//
// Decision quantities (E, M, B, the region set and its integer moments) are
// computed in FP64 / exact integers; this file is compiled with
// -ffp-contract=off.  Connected components use a lock-free union-find whose
// roots are always the smallest pixel index of their component, so labels are
// canonical and independent of thread scheduling: first inside 16x16 tiles in
// LDS (fused with the classification and the erosion), then across tile
// borders in global memory.  Kept regions take their record slots from the
// counts of the pixel chunks before theirs, so records stay in ascending
// (view, label) order.
//
// Every kernel covers the views of one call together (one view, or a batch):
// a view of a megapixel keeps the chip busy for a few microseconds per pass,
// less than a launch costs, so view by view the passes were launch-bound
// (16 views of 1256x828: 70 us a view, 1120 us; 375 us in two batches of eight).
#include <mutex>

#include "internal.h"

namespace {

constexpr int ES_MAX_BATCH = AS_MAX_VIEWS;   // views of one call

enum { ES_B, ES_LABEL, ES_MOM, ES_BASE, ES_KIDX, ES_COUNT };

// Pixels per block of the pass that counts kept regions (four consecutive ones
// a thread), and blocks that write a chunk's records.
constexpr int ES_CHUNK = 4096;
constexpr int ES_PARTS = 4;

// Bytes of each scratch slot for views of P pixels in all (each view's pixels
// rounded up to a multiple of four): bands, labels, the six integer moments
// per (root) pixel, the record count on entry, and a word per chunk of pixels
// (each view's last one may be partial).
void es_need(int64_t P, size_t need[ES_COUNT]) {
    const size_t p = (size_t)(P > 0 ? P : 1);
    need[ES_B] = p;
    need[ES_LABEL] = p * 4;
    need[ES_MOM] = p * 48;
    need[ES_BASE] = 8;
    need[ES_KIDX] = ((p + ES_CHUNK - 1) / ES_CHUNK + ES_MAX_BATCH) * 8;
}

// One view of a call.  Its pixels, 16x16 tiles and chunks of ES_CHUNK pixels
// are [pix0, ..), [tile0, ..) and [chunk0, ..) of the call's.
struct EsView {
    const double *err;
    const unsigned long long *minmax;
    const int32_t *dom;
    const float *gt;
    int64_t pix0;
    int32_t W, H, tiles_x, tile0, chunk0, id;
};
// The views of a call, passed to each of its kernels by value.  A call of one
// view, which is what a view-by-view loop makes, has a table of one: with the
// table of ES_MAX_BATCH (1 KB to write for each of the five launches) the first
// error map and statistics of a 1256x828 view on a new context took 201 to
// 220 us, with this one 119 to 125 (the arguments' memory is cold then), and
// later ones 73 against 71 us.
template <int CAP>
struct EsBatch {
    int32_t n, tiles, chunks;
    EsView v[CAP];
};
template <int CAP>
__device__ __forceinline__ const EsView &view_of_es_tile(const EsBatch<CAP> &b, int tile) {
    if (CAP == 1) return b.v[0];
    int k = 0;
    for (int q = 1; q < b.n; q++) k += tile >= b.v[q].tile0 ? 1 : 0;
    return b.v[k];
}
template <int CAP>
__device__ __forceinline__ const EsView &view_of_es_chunk(const EsBatch<CAP> &b, int chunk) {
    if (CAP == 1) return b.v[0];
    int k = 0;
    for (int q = 1; q < b.n; q++) k += chunk >= b.v[q].chunk0 ? 1 : 0;
    return b.v[k];
}

__device__ __forceinline__ double dev_bits_to_double(unsigned long long b) { return __longlong_as_double((long long)b); }

// Per-pixel L1 error and its range.  A bounded grid strides over the pixels
// and each block issues one pair of range atomics: device-wide atomics on the
// same two words serialise at the memory side, so there are few of them.
constexpr int EM_THREADS = 1024;
__global__ void __launch_bounds__(EM_THREADS) k_error_map(int W, int H, const float *__restrict__ img,
                                                   const float *__restrict__ gt, double *__restrict__ err,
                                                   unsigned long long *__restrict__ minmax) {
    __shared__ double s_mn[EM_THREADS / 64], s_mx[EM_THREADS / 64];
    const int64_t P = (int64_t)W * H;
    double mn = __longlong_as_double(0x7ff0000000000000ll), mx = 0.0;
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < P; u += (int64_t)gridDim.x * blockDim.x) {
        const double d0 = fabs((double)img[u] - (double)gt[u]);
        const double d1 = fabs((double)img[P + u] - (double)gt[P + u]);
        const double d2 = fabs((double)img[2 * P + u] - (double)gt[2 * P + u]);
        const double e = (d0 + d1) + d2;
        err[u] = e;
        mn = fmin(mn, e);
        mx = fmax(mx, e);
    }
    mn = wave_min_d(mn);
    mx = wave_max_d(mx);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_mn[w] = mn;
        s_mx[w] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < EM_THREADS / 64; k++) {
            mn = fmin(mn, s_mn[k]);
            mx = fmax(mx, s_mx[k]);
        }
        atomicMin(&minmax[0], (unsigned long long)__double_as_longlong(mn));
        atomicMax(&minmax[1], (unsigned long long)__double_as_longlong(mx));
    }
}

__global__ void k_error_map_init(unsigned long long *__restrict__ minmax) {
    minmax[0] = 0x7ff0000000000000ull;
    minmax[1] = 0ull;
}

// E = normalised error (Eq. (l1map)), M = [E > tau], band B = floor((E - tau) L / (1 - tau)) clamped to L - 1
__device__ __forceinline__ bool classify_px(double e, double emin, double emax, double tau, int L, uint8_t *band) {
    const double E = (emax == emin) ? 0.0 : (e - emin) / (emax - emin);
    const bool m = E > tau;
    uint8_t b = 0;
    if (m) {
        double bb = floor(((E - tau) * (double)L) / (1.0 - tau));
        if (bb > (double)(L - 1)) bb = (double)(L - 1);
        b = (uint8_t)bb;
    }
    *band = b;
    return m;
}

__device__ __forceinline__ int32_t uf_load(const int32_t *L, int32_t x) {
    return __hip_atomic_load(L + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t uf_find(const int32_t *L, int32_t x) {
    int32_t p = uf_load(L, x);
    while (p != x) {
        x = p;
        p = uf_load(L, x);
    }
    return x;
}

// Link the components of a and b; a root only ever points to a smaller index.
__device__ __forceinline__ void uf_unite(int32_t *L, int32_t a, int32_t b) {
    while (true) {
        a = uf_find(L, a);
        b = uf_find(L, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicMin(L + a, b);
        if (old == a) return;
        a = old;
    }
}

// The same union-find on a block's LDS array.
__device__ __forceinline__ int lds_find(int32_t *L, int x) {
    int p = __hip_atomic_load(L + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (p != x) {
        x = p;
        p = __hip_atomic_load(L + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return x;
}

__device__ __forceinline__ void lds_unite(int32_t *L, int a, int b) {
    while (true) {
        a = lds_find(L, a);
        b = lds_find(L, b);
        if (a == b) return;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(L + a, b);
        if (old == a) return;
        a = old;
    }
}

constexpr int ET = 16;      // pixel tile of the erosion / local components
constexpr int EMAX_R = 8;   // erosion radii up to this use an LDS tile with halo
constexpr int ES = ET + 2 * EMAX_R;

// The smallest error that classify_px puts above tau, so that the halo
// pixels take a compare instead of a division each: (e - emin) / (emax - emin)
// rounds monotonically in e for a positive finite range, so {E > tau} is
// {e >= threshold}.  Found by stepping from emin + tau (emax - emin), which is
// within a few ulps of it.  False when there is no such threshold (an empty
// or non-finite range, or a caller's range turned round): classify directly.
__device__ bool error_threshold(double emin, double emax, double tau, double *thr) {
    const double d = emax - emin;
    if (!(d > 0.0) || !(d < __longlong_as_double(0x7ff0000000000000ll))) return false;
    double c = emin + tau * d;
    if (!(c >= 0.0)) return false;
    int step = 0;
    for (; step < 64 && !((c - emin) / d > tau); step++) c = __longlong_as_double(__double_as_longlong(c) + 1);
    for (; step < 64 && c > 0.0; step++) {
        const double below = __longlong_as_double(__double_as_longlong(c) - 1);
        if (!((below - emin) / d > tau)) break;
        c = below;
    }
    *thr = c;
    return step < 64;
}

// M' = erosion of M with a square element of offsets [-lo, hi] per axis
// ((2r+1)^2: lo = hi = r; pixels outside the image count as set); active = M'
// and a candidate dominates the pixel.  Then the
// 8-connected components of equal (D, B) inside the block's 16x16 tile, with
// an LDS union-find whose roots are the smallest tile-local index, which is
// also the smallest image index of the tile's part of the component.  Writes
// label = image index of that root (-1 inactive) and, at active pixels, the
// band.  A tile without a high-error pixel of a candidate stops after its own
// pixels: the element holds the pixel itself, so nothing in it can be active.
template <int CAP>
__global__ void __launch_bounds__(ET * ET) k_erode_ccl_local(const EsBatch<CAP> eb, int r, int lo, int hi, double tau,
                                                             int L, uint8_t *__restrict__ B_all,
                                                             const uint8_t *__restrict__ is_cand,
                                                             int32_t *__restrict__ attr,
                                                             int32_t *__restrict__ label_all,
                                                             unsigned long long *__restrict__ mom_all) {
    __shared__ uint8_t s_m[ES * ES];
    __shared__ uint8_t s_row[ES * ET];
    __shared__ int32_t s_par[ET * ET];
    __shared__ int32_t s_dom[ET * ET];
    __shared__ uint8_t s_b[ET * ET];
    __shared__ double s_thr;
    __shared__ int s_has_thr;
    const EsView &ev = view_of_es_tile(eb, (int)blockIdx.x);
    const int W = ev.W, H = ev.H;
    const double *__restrict__ err = ev.err;
    uint8_t *B = B_all + ev.pix0;
    int32_t *label = label_all + ev.pix0;
    unsigned long long *mom = mom_all + 6 * ev.pix0;
    const int tid = threadIdx.x;
    const int tile = (int)blockIdx.x - ev.tile0;
    const int tx = tile % ev.tiles_x, ty = tile / ev.tiles_x;
    const int ox = tx * ET, oy = ty * ET;
    const int lx = tid % ET, ly = tid / ET, x = ox + lx, y = oy + ly;
    const bool inside = x < W && y < H;
    const int64_t u = (int64_t)y * W + x;
    const double emin = dev_bits_to_double(ev.minmax[0]), emax = dev_bits_to_double(ev.minmax[1]);
    uint8_t scratch_band;
    // this pixel's class and band, and the attribution count before erosion:
    // attr[D] += 1 per high-error pixel dominated by a candidate, one atomic
    // per wave when all hits share D
    uint8_t b = 0;
    const int32_t d = inside ? ev.dom[u] : -1;
    const bool m_own = inside && classify_px(err[u], emin, emax, tau, L, &b);
    const bool hit = m_own && d >= 0 && is_cand[d];
    {
        const uint64_t hits = __ballot(hit);
        if (hits) {
            const int leader = __ffsll((unsigned long long)hits) - 1;
            const int32_t d0 = __shfl(d, leader, 64);
            const uint64_t same = __ballot(hit && d == d0);
            if (same == hits) {
                if ((int)__lane_id() == leader) atomicAdd(&attr[d0], (int32_t)__popcll(hits));
            } else if (hit) {
                atomicAdd(&attr[d], 1);
            }
        }
    }
    if (!__syncthreads_or(hit)) {
        if (inside) label[u] = -1;
        return;
    }
    bool e;
    if (r <= EMAX_R) {   // lo, hi <= r
        if (tid == 0) s_has_thr = error_threshold(emin, emax, tau, &s_thr) ? 1 : 0;
        const int S = ET + lo + hi;
        double h[(ES * ES) / (ET * ET)];   // the halo's errors, loaded before the threshold is known
#pragma unroll
        for (int q = 0; q < (ES * ES) / (ET * ET); q++) {
            const int i = tid + q * ET * ET;
            const int hx = i % S, hy = i / S, gx = ox + hx - lo, gy = oy + hy - lo;
            h[q] = 0.0;
            if (i < S * S && gx >= 0 && gy >= 0 && gx < W && gy < H) h[q] = err[(int64_t)gy * W + gx];
        }
        __syncthreads();
        const bool has_thr = s_has_thr != 0;
        const double thr = s_thr;
#pragma unroll
        for (int q = 0; q < (ES * ES) / (ET * ET); q++) {
            const int i = tid + q * ET * ET;
            if (i >= S * S) break;
            const int hx = i % S, hy = i / S, gx = ox + hx - lo, gy = oy + hy - lo;
            s_m[i] = (gx < 0 || gy < 0 || gx >= W || gy >= H)
                         ? 1
                         : (has_thr ? h[q] >= thr : classify_px(h[q], emin, emax, tau, L, &scratch_band));
        }
        __syncthreads();
        for (int i = tid; i < S * ET; i += ET * ET) {   // AND along rows
            const int cx = i % ET, hy = i / ET;
            uint8_t a = 1;
            for (int k = 0; k <= lo + hi; k++) a &= s_m[hy * S + cx + k];
            s_row[i] = a;
        }
        __syncthreads();
        uint8_t a = 1;                                  // then along columns
        for (int k = 0; k <= lo + hi; k++) a &= s_row[(ly + k) * ET + lx];
        e = a != 0;
    } else {
        e = m_own;
        for (int dy = -lo; dy <= hi && e; dy++) {
            const int yy = y + dy;
            if (yy < 0 || yy >= H) continue;
            for (int dx = -lo; dx <= hi; dx++) {
                const int xx = x + dx;
                if (xx < 0 || xx >= W) continue;
                if (!classify_px(err[(int64_t)yy * W + xx], emin, emax, tau, L, &scratch_band)) {
                    e = false;
                    break;
                }
            }
        }
    }
    const bool active = inside && e && d >= 0 && is_cand[d];
    s_par[tid] = active ? tid : -1;
    s_dom[tid] = d;
    s_b[tid] = b;
    __syncthreads();
    if (active) {
        const int nx[4] = {-1, -1, 0, 1};
        const int ny[4] = {0, -1, -1, -1};
        for (int k = 0; k < 4; k++) {
            const int qx = lx + nx[k], qy = ly + ny[k];
            if (qx < 0 || qy < 0 || qx >= ET) continue;
            const int q = qy * ET + qx;
            if (s_par[q] < 0 || s_dom[q] != d || s_b[q] != b) continue;   // activity never changes here
            lds_unite(s_par, tid, q);
        }
    }
    __syncthreads();
    if (inside) {
        int32_t lab = -1;
        if (active) {
            B[u] = b;
            const int rt = lds_find(s_par, tid);
            lab = (int32_t)((int64_t)(oy + rt / ET) * W + ox + rt % ET);
            // every component's final root (its smallest index) is the local
            // root of its part in that tile: the moments are cleared there
            if (rt == tid)
                for (int k = 0; k < 6; k++) mom[u * 6 + k] = 0ull;
        }
        label[u] = lab;
    }
}

// Join the tile-local components across tile borders: only pixels whose W,
// NW, N or NE neighbour lies in another tile link (a tile's top row, left
// and right columns: 3 ET - 2 pixels, one thread each), with the global
// union-find (roots are the smallest image index).
constexpr int ES_BORDER = 3 * ET - 2;
template <int CAP>
__global__ void k_ccl_border(const EsBatch<CAP> eb, const uint8_t *__restrict__ B_all, int32_t *label_all) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)eb.tiles * ES_BORDER) return;
    const int64_t gt = i / ES_BORDER;
    const int j = (int)(i - gt * ES_BORDER);
    const EsView &ev = view_of_es_tile(eb, (int)gt);
    const int W = ev.W, H = ev.H, t = (int)gt - ev.tile0;
    const int32_t *__restrict__ dom = ev.dom;
    const uint8_t *B = B_all + ev.pix0;
    int32_t *label = label_all + ev.pix0;
    // j < ET: top row; then the left and the right column below it
    const int lx = j < ET ? j : (j < 2 * ET - 1 ? 0 : ET - 1);
    const int ly = j < ET ? 0 : (j < 2 * ET - 1 ? j - ET + 1 : j - 2 * ET + 2);
    const int x = (t % ev.tiles_x) * ET + lx, y = (t / ev.tiles_x) * ET + ly;
    if (x >= W || y >= H) return;
    const int64_t u = (int64_t)y * W + x;
    // a label's sign (active or not) never changes in this pass, only the
    // values of roots do: plain loads decide activity, the union-find reads
    // coherently
    const volatile int32_t *lv = label;
    if (lv[u] < 0) return;
    const int32_t d = dom[u];
    const uint8_t b = B[u];
    const int nx[4] = {-1, -1, 0, 1};
    const int ny[4] = {0, -1, -1, -1};
    for (int k = 0; k < 4; k++) {
        const int xx = x + nx[k], yy = y + ny[k];
        if (xx < 0 || yy < 0 || xx >= W) continue;
        if (xx / ET == x / ET && yy / ET == y / ET) continue;   // joined by the local pass
        const int64_t q = (int64_t)yy * W + xx;
        if (lv[q] < 0 || dom[q] != d || B[q] != b) continue;    // an inactive pixel's band is not written
        uf_unite(label, (int32_t)u, (int32_t)q);
    }
}

// Exact integer moments A, Sx, Sy, Sxx, Sxy, Syy per component, stored at the
// component's root pixel (the end of the pixel's parent chain: the labels no
// longer change, so plain loads follow it).  One block per tile, one set of
// atomics per distinct region among a wave's 64 pixels (four row segments of a
// tile, which few regions of a smooth error map cross).  A noisy one has tens
// of regions in a wave, one after another, so a region's sums are short: taken
// about the wave's first pixel they fit two words of three fields (at most 64,
// 480 and 4960; 96, 720 and 224), which two DPP sums give and integer
// arithmetic moves to the image's origin.  As six 64-bit sums by lane
// exchanges a noisy 172x248 view took 41 us (22 with rows of 64 pixels a wave,
// as the pass once had), one of 244x183 40; now 13 and 12.
template <int CAP>
__global__ void __launch_bounds__(ET * ET) k_moments(const EsBatch<CAP> eb, const int32_t *__restrict__ label_all,
                                                     unsigned long long *__restrict__ mom_all) {
    static_assert(ET == 16, "the fields' widths");
    const EsView &ev = view_of_es_tile(eb, (int)blockIdx.x);
    const int32_t *label = label_all + ev.pix0;
    unsigned long long *mom = mom_all + 6 * ev.pix0;
    const int tile = (int)blockIdx.x - ev.tile0;
    const int lane = (int)__lane_id();
    const uint32_t lx = (uint32_t)lane & 15, ly = (uint32_t)lane >> 4;
    const int64_t X = (int64_t)(tile % ev.tiles_x) * ET;
    const int64_t Y = (int64_t)(tile / ev.tiles_x) * ET + (threadIdx.x >> 6) * 4;
    int32_t s = -1;
    if (X + lx < ev.W && Y + ly < ev.H) {
        int32_t l = label[(Y + ly) * ev.W + X + lx];
        if (l >= 0) {
            for (int32_t p = label[l]; p != l; p = label[l]) l = p;
            s = l;
        }
    }
    const uint32_t vx = 1u | lx << 7 | lx * lx << 16, vy = ly | lx * ly << 8 | ly * ly << 20;
    uint64_t pending = __ballot(s >= 0);
    while (pending) {
        const int leader = __ffsll((unsigned long long)pending) - 1;
        const int32_t s0 = __builtin_amdgcn_readlane(s, leader);
        const bool mine = s == s0;
        pending &= ~__ballot(mine);
        const uint32_t tx = last_lane(wave_prefix(mine ? vx : 0u)), ty = last_lane(wave_prefix(mine ? vy : 0u));
        const int64_t A = tx & 127, sx = tx >> 7 & 511, sxx = tx >> 16;
        const int64_t sy = ty & 255, sxy = ty >> 8 & 4095, syy = ty >> 20;
        int64_t t = A;
        if (lane == 1) t = A * X + sx;
        if (lane == 2) t = A * Y + sy;
        if (lane == 3) t = (A * X + 2 * sx) * X + sxx;
        if (lane == 4) t = (A * Y + sy) * X + sx * Y + sxy;
        if (lane == 5) t = (A * Y + 2 * sy) * Y + syy;
        if (lane < 6) atomicAdd(&mom[(int64_t)s0 * 6 + lane], (unsigned long long)t);
    }
}

// The kept components (Eq. (min_region_area)) among a thread's four pixels of
// a chunk: bit j for pixel u + j, a root whose area is at least m_min.
__device__ __forceinline__ uint32_t kept_bits(const EsView &ev, const int32_t *label, const unsigned long long *mom,
                                              int64_t u, int m_min) {
    const int64_t P = (int64_t)ev.W * ev.H;
    if (u >= P) return 0u;
    // the chunk's labels are 16-byte aligned (pix0 is a multiple of four) and
    // the slot holds each view's pixels rounded up to a multiple of four
    const int4 l = *reinterpret_cast<const int4 *>(label + u);
    const int32_t lab[4] = {l.x, l.y, l.z, l.w};
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < 4; j++)
        if (u + j < P && lab[j] == (int32_t)(u + j) && (int64_t)mom[(u + j) * 6] >= (int64_t)m_min) bits |= 1u << j;
    return bits;
}

// Kept components per chunk (the low 16 bits of its word; above them, those
// before its second, third and fourth part); the first block also notes the
// records already in the buffer, which the next pass counts on while it
// advances the count.
template <int CAP>
__global__ void __launch_bounds__(ES_CHUNK / 4) k_region_keep(const EsBatch<CAP> eb, const int32_t *__restrict__ label_all,
                                                              const unsigned long long *__restrict__ mom_all, int m_min,
                                                              const int64_t *__restrict__ count,
                                                              int64_t *__restrict__ base, int64_t *__restrict__ part) {
    __shared__ int s_w[ES_CHUNK / 256];
    const EsView &ev = view_of_es_chunk(eb, (int)blockIdx.x);
    const int64_t u = (int64_t)((int)blockIdx.x - ev.chunk0) * ES_CHUNK + 4 * (int64_t)threadIdx.x;
    int c = __popc(kept_bits(ev, label_all + ev.pix0, mom_all + 6 * ev.pix0, u, m_min));
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        constexpr int WAVES = ES_CHUNK / 256 / ES_PARTS;   // of a part
        uint64_t word = 0;
        for (int k = 1; k < ES_CHUNK / 256; k++) {
            if (k % WAVES == 0) word |= (uint64_t)c << 16 * (k / WAVES);
            c += s_w[k];
        }
        part[blockIdx.x] = (int64_t)(word | (uint64_t)c);
        if (blockIdx.x == 0) *base = *count;
    }
}

__device__ __forceinline__ double central_moment(int64_t A, int64_t sab, int64_t sa, int64_t sb) {
    const __int128 num = (__int128)A * sab - (__int128)sa * sb;
    double dnum;
    if (num >= (__int128)INT64_MIN && num <= (__int128)INT64_MAX) dnum = (double)(int64_t)num;
    else dnum = (double)num;
    const double dA = (double)A;
    return dnum / (dA * dA);
}

// One record per kept component, in ascending (view, label) order.  A block
// sums the chunk counts before its own (a few loads a thread, less than a
// launch of a scan between the passes) and the last one advances the buffer's
// count.  A record is a long chain in FP64, so what bounds a view of few
// pixels is the records that fall to one thread and to one CU: a block has a
// quarter of a chunk, and its kept pixels are listed in LDS for the threads to
// take one each.  With a block for a chunk and a thread's records left to it, a
// noisy 244x183 view took 19 us, now 7.
template <int CAP>
__global__ void __launch_bounds__(ES_CHUNK / ES_PARTS / 4)
k_region_emit(const EsBatch<CAP> eb, const int32_t *__restrict__ label_all,
              const unsigned long long *__restrict__ mom_all, int m_min, const uint8_t *__restrict__ B_all,
              const int64_t *__restrict__ base, const int64_t *__restrict__ part, as_region *__restrict__ out,
              int64_t out_cap, int64_t *__restrict__ count) {
    constexpr int PX = ES_CHUNK / ES_PARTS, THREADS = PX / 4, NW = THREADS / 64;
    static_assert(ES_PARTS == 4 && ES_CHUNK < 65536, "a chunk's word");
    __shared__ int64_t s_pre[NW];
    __shared__ int s_w[NW];
    __shared__ uint16_t s_kept[PX];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int blk = (int)blockIdx.x / ES_PARTS, q = (int)blockIdx.x % ES_PARTS;
    const EsView &ev = view_of_es_chunk(eb, blk);
    const int32_t *label = label_all + ev.pix0;
    const unsigned long long *mom = mom_all + 6 * ev.pix0;
    const int64_t u0 = (int64_t)(blk - ev.chunk0) * ES_CHUNK + q * PX;
    int64_t pre = 0;
    for (int b = (int)threadIdx.x; b < blk; b += THREADS) pre += part[b] & 0xffff;
    for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o, 64);
    const uint32_t bits = kept_bits(ev, label, mom, u0 + 4 * (int64_t)threadIdx.x, m_min);
    const int own = __popc(bits);
    const int inc = (int)wave_prefix((uint32_t)own);
    if (lane == 63) s_w[w] = inc;
    if (lane == 0) s_pre[w] = pre;
    __syncthreads();
    int kept = 0, at = inc - own;
    int64_t first = *base;
    for (int k = 0; k < NW; k++) {
        first += s_pre[k];
        kept += s_w[k];
        at += k < w ? s_w[k] : 0;
    }
    const uint64_t word = (uint64_t)part[blk];
    if ((int)blockIdx.x == (int)gridDim.x - 1 && threadIdx.x == 0) *count = first + (int64_t)(word & 0xffff);
    if (q > 0) first += (int64_t)(word >> 16 * q & 0xffff);
    for (uint32_t left = bits; left; left &= left - 1) s_kept[at++] = (uint16_t)(4 * threadIdx.x + __ffs((int)left) - 1);
    __syncthreads();
    const int W = ev.W;
    const int64_t P = (int64_t)W * ev.H;
    const uint8_t *B = B_all + ev.pix0;
    for (int k = (int)threadIdx.x; k < kept; k += THREADS) {
        const int64_t s = u0 + s_kept[k];
        const int64_t pos = first + k;
        if (pos >= out_cap) return;
        as_region r;
        const int32_t root = (int32_t)s;
        r.cand = ev.dom[root];
        r.view = ev.id;
        r.label = root;
        r.band = B[root];
        r.pad0 = 0;
        const int64_t A = (int64_t)mom[s * 6 + 0];
        r.area = (int32_t)A;
        r.sx = (int64_t)mom[s * 6 + 1];
        r.sy = (int64_t)mom[s * 6 + 2];
        r.sxx = (int64_t)mom[s * 6 + 3];
        r.sxy = (int64_t)mom[s * 6 + 4];
        r.syy = (int64_t)mom[s * 6 + 5];
        const double dA = (double)A;
        r.cx = (double)r.sx / dA + 0.5;
        r.cy = (double)r.sy / dA + 0.5;
        const double cxx = central_moment(A, r.sxx, r.sx, r.sx) + 1.0 / 12.0;
        const double cxy = central_moment(A, r.sxy, r.sx, r.sy);
        const double cyy = central_moment(A, r.syy, r.sy, r.sy) + 1.0 / 12.0;
        r.cov[0] = cxx;
        r.cov[1] = cxy;
        r.cov[2] = cyy;
        const double half_tr = 0.5 * (cxx + cyy);
        const double half_dif = 0.5 * (cxx - cyy);
        const double disc = sqrt(half_dif * half_dif + cxy * cxy);
        const double l1 = half_tr + disc, l2 = half_tr - disc;
        double ex, ey;
        if (disc == 0.0) {
            ex = 1.0; ey = 0.0;
        } else if (half_dif >= 0.0) {
            ex = half_dif + disc; ey = cxy;
        } else {
            ex = cxy; ey = -half_dif + disc;
        }
        const double en = sqrt(ex * ex + ey * ey);
        ex = ex / en;
        ey = ey / en;
        if (ex < 0.0 || (ex == 0.0 && ey < 0.0)) {
            ex = -ex;
            ey = -ey;
        }
        r.e1[0] = ex;
        r.e1[1] = ey;
        r.sigma1 = sqrt(l1);
        r.sigma2 = sqrt(l2 > 0.0 ? l2 : 0.0);
        const int64_t gx = (int64_t)floor(r.cx), gy = (int64_t)floor(r.cy);
        for (int ch = 0; ch < 3; ch++) r.rgb[ch] = ev.gt[ch * P + gy * W + gx];
        r.pad1 = 0.f;
        out[pos] = r;
    }
}


}  // namespace

void launch_error_map(int W, int H, const float *image, const float *gt, double *err, uint64_t *minmax, hipStream_t s) {
    const int64_t P = (int64_t)W * H;
    hipLaunchKernelGGL(k_error_map_init, dim3(1), dim3(1), 0, s, reinterpret_cast<unsigned long long *>(minmax));
    if (P == 0) return;
    int64_t g = (P + EM_THREADS - 1) / EM_THREADS;
    if (g > 256) g = 256;
    hipLaunchKernelGGL(k_error_map, dim3((unsigned)g), dim3(EM_THREADS), 0, s, W, H, image, gt, err,
                       reinterpret_cast<unsigned long long *>(minmax));
}

size_t errstats_reserve_bytes(int64_t max_pixels) {
    if (max_pixels <= 0) return 0;
    size_t need[ES_COUNT], total = 0;
    es_need(max_pixels, need);
    for (int k = 0; k < ES_COUNT; k++) total += devbuf_size(need[k]);
    return total;
}

hipError_t errstats_reserve(as_ctx *ctx, int64_t max_pixels) {
    if (max_pixels <= 0) return hipSuccess;
    size_t need[ES_COUNT];
    es_need(max_pixels, need);
    hipError_t e = hipSuccess;
    for (int k = 0; k < ES_COUNT && e == hipSuccess; k++) e = devbuf_ensure(ctx->es[k], need[k]);
    return e;
}

namespace {
// The scratch of one error-statistics call (slots of es_need).
struct EsScratch {
    uint8_t *B;
    int32_t *label;
    unsigned long long *mom;
    int64_t *base;   // the record count on entry
    int64_t *part;   // per chunk of pixels: kept components
};

template <int CAP>
void es_launch(const EsScratch &sc, const EsBatch<CAP> &eb, const uint8_t *is_cand, const as_split_params &p,
               as_region_buf &rb, int32_t *attr, hipStream_t s);

// The kernels' view table; returns the pixels the scratch has to hold.
template <int CAP>
int64_t es_batch(int n, const as_error_view *views, EsBatch<CAP> &eb) {
    int64_t pix = 0, tiles = 0, chunks = 0;
    for (int k = 0; k < n; k++) {
        const as_error_view &a = views[k];
        const int64_t P = (int64_t)a.width * a.height;
        EsView &v = eb.v[k];
        v.err = a.err;
        v.minmax = reinterpret_cast<const unsigned long long *>(a.err_minmax);
        v.dom = a.dom;
        v.gt = a.gt;
        v.pix0 = (pix + 3) & ~(int64_t)3;
        v.W = a.width;
        v.H = a.height;
        v.tiles_x = (a.width + ET - 1) / ET;
        v.tile0 = (int32_t)tiles;
        v.chunk0 = (int32_t)chunks;
        v.id = a.view_id;
        pix = v.pix0 + P;
        tiles += (int64_t)v.tiles_x * ((a.height + ET - 1) / ET);
        chunks += (P + ES_CHUNK - 1) / ES_CHUNK;
    }
    eb.n = n;
    eb.tiles = (int32_t)tiles;
    eb.chunks = (int32_t)chunks;
    return pix;
}
}  // namespace

as_status run_error_stats(as_ctx *ctx, int n_views, const as_error_view *views, const uint8_t *is_cand,
                          const as_split_params &p, as_region_buf &rb, int32_t *attr, hipStream_t s) {
    EsBatch<1> one;
    EsBatch<ES_MAX_BATCH> many;
    const int64_t pix = n_views == 1 ? es_batch(1, views, one) : es_batch(n_views, views, many);
    if (pix > ctx->res.max_pixels) {
        as_set_error("as_accumulate_error_stats: %d view%s (the first %dx%d) need max_pixels >= %lld in as_ctx_reserve "
                     "(reserved %lld)", n_views, n_views == 1 ? "" : "s", views[0].width, views[0].height,
                     (long long)pix, (long long)ctx->res.max_pixels);
        return AS_ERR_CAPACITY;
    }
    DevBuf *es = ctx->es;
    const EsScratch sc{(uint8_t *)es[ES_B].p, (int32_t *)es[ES_LABEL].p, (unsigned long long *)es[ES_MOM].p,
                       (int64_t *)es[ES_BASE].p, (int64_t *)es[ES_KIDX].p};
    if (n_views == 1) es_launch(sc, one, is_cand, p, rb, attr, s);
    else es_launch(sc, many, is_cand, p, rb, attr, s);
    return AS_OK;
}

// ---- the no-allocation variant ------------------------------------------------------
//
// For callers that cannot allocate device memory (code under graph capture,
// serving loops, harnesses that forbid hipMalloc): the same kernels with their
// scratch in one static device array, sized for views of up to
// AS_NOALLOC_MAX_PIXELS pixels.  The runtime gives every device its own copy
// of the array (held until the process ends); its address on a device is taken
// once, with that device current, when a context is created there
// (errstats_noalloc_init), and the kernels receive that address.  In host code
// the array's name is no device address, so it is never passed to a kernel.
// Every call on a device shares the one array: calls on that device must not
// overlap (they would race on it).  Nothing in it needs clearing: each kernel
// writes a slot before any kernel of the same call reads it.
namespace {
constexpr size_t es_slot(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
constexpr size_t ES_NA_PIX = (size_t)AS_NOALLOC_MAX_PIXELS;
constexpr size_t ES_NA_OFF_LABEL = es_slot(ES_NA_PIX);
constexpr size_t ES_NA_OFF_MOM = ES_NA_OFF_LABEL + es_slot(ES_NA_PIX * 4);
constexpr size_t ES_NA_OFF_BASE = ES_NA_OFF_MOM + es_slot(ES_NA_PIX * 48);
constexpr size_t ES_NA_OFF_KIDX = ES_NA_OFF_BASE + es_slot(8);
constexpr size_t ES_NA_BYTES = ES_NA_OFF_KIDX + es_slot((ES_NA_PIX + ES_CHUNK - 1) / ES_CHUNK * 8);
constexpr int ES_NA_MAX_DEVICES = 64;

std::mutex g_na_mutex;
unsigned char *g_na_ptr[ES_NA_MAX_DEVICES];   // the array's address on each device
}  // namespace

static __device__ __align__(256) unsigned char scratch[ES_NA_BYTES];

hipError_t errstats_noalloc_init(int device) {
    if (device < 0 || device >= ES_NA_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_na_mutex);
    if (g_na_ptr[device]) return hipSuccess;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_na_ptr[device] = (unsigned char *)ptr;
    return hipSuccess;
}

size_t errstats_noalloc_bytes() { return ES_NA_BYTES; }

as_status run_error_stats_noalloc(as_ctx *ctx, const as_error_view &view, const uint8_t *is_cand,
                                  const as_split_params &p, as_region_buf &rb, int32_t *attr, hipStream_t s) {
    const int W = view.width, H = view.height;
    const int64_t P = (int64_t)W * H;
    if (P > (int64_t)AS_NOALLOC_MAX_PIXELS) {
        as_set_error("as_accumulate_error_stats_noalloc: a %dx%d view has %lld pixels, above the static scratch's "
                     "maximum of %lld", W, H, (long long)P, (long long)AS_NOALLOC_MAX_PIXELS);
        return AS_ERR_CAPACITY;
    }
    unsigned char *base = nullptr;
    if (ctx->device >= 0 && ctx->device < ES_NA_MAX_DEVICES) {
        std::lock_guard<std::mutex> lock(g_na_mutex);
        base = g_na_ptr[ctx->device];
    }
    if (!base) {
        as_set_error("as_accumulate_error_stats_noalloc: no static scratch address for device %d", ctx->device);
        return AS_ERR_STATE;
    }
    const EsScratch sc{base, (int32_t *)(base + ES_NA_OFF_LABEL), (unsigned long long *)(base + ES_NA_OFF_MOM),
                       (int64_t *)(base + ES_NA_OFF_BASE), (int64_t *)(base + ES_NA_OFF_KIDX)};
    EsBatch<1> eb;
    es_batch(1, &view, eb);
    es_launch(sc, eb, is_cand, p, rb, attr, s);
    return AS_OK;
}

namespace {
template <int CAP>
void es_launch(const EsScratch &sc, const EsBatch<CAP> &eb, const uint8_t *is_cand, const as_split_params &p,
               as_region_buf &rb, int32_t *attr, hipStream_t s) {
    // element offsets: [-r, r] per axis, or a side of r + 1 (flag)
    const int lo = (p.flags & AS_SPLIT_ERODE_SIDE) ? p.r_erode / 2 : p.r_erode;
    const int hi = (p.flags & AS_SPLIT_ERODE_SIDE) ? p.r_erode - p.r_erode / 2 : p.r_erode;
    const dim3 tiles((unsigned)eb.tiles), chunks((unsigned)eb.chunks), cb(ES_CHUNK / 4);
    // classification, attribution, erosion and the tile-local components in one pass
    hipLaunchKernelGGL(k_erode_ccl_local<CAP>, tiles, dim3(ET * ET), 0, s, eb, p.r_erode, lo, hi, p.tau_l1, p.L, sc.B,
                       is_cand, attr, sc.label, sc.mom);
    const int64_t nb = ((int64_t)eb.tiles * ES_BORDER + 255) / 256;
    hipLaunchKernelGGL(k_ccl_border<CAP>, dim3((unsigned)nb), dim3(256), 0, s, eb, sc.B, sc.label);
    hipLaunchKernelGGL(k_moments<CAP>, tiles, dim3(ET * ET), 0, s, eb, sc.label, sc.mom);
    // kept roots per chunk, then their records (advancing the buffer's count)
    hipLaunchKernelGGL(k_region_keep<CAP>, chunks, cb, 0, s, eb, sc.label, sc.mom, p.m_min, rb.count, sc.base, sc.part);
    hipLaunchKernelGGL(k_region_emit<CAP>, dim3(chunks.x * ES_PARTS), dim3(ES_CHUNK / ES_PARTS / 4), 0, s, eb, sc.label,
                       sc.mom, p.m_min, sc.B, sc.base, sc.part, rb.records, rb.capacity, rb.count);
}
}  // namespace

AS_WARM_KERNEL(errstats)
