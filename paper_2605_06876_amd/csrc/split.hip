// The AdpSplit adaptive split (Sec. 4.2, 4.3, App. A and the implementation
// details of Sec. 5) and the stream-compacted append.
//
//   1. region records sorted by (candidate, view, label) with the LDS radix
//      sorter, so that each candidate owns a contiguous range;
//   2. one thread per region: child proposal (centre at t* of Eq. (tstar) on
//      the centroid ray, shape from the clipped, unprojected PCA axes,
//      Gram-Schmidt rotation [u1 | u2 | z_v], colour from the target);
//   3. one wave per region, three launches: transitive merge graph under
//      Eq. (merge_conditions) (lock-free union-find, roots = first member),
//      merged parameters of Eq. (merge_cov), ranking by covariance extent and
//      the N_max cap; then one thread per candidate: the mode (vanilla / reset
//      / adaptive / random) and count (the ablation variants of Table 2 skip
//      the merge, or the region children altogether);
//   4. scans of the counts and of the removal mask, survivor copy and child
//      write-out.
// All decision arithmetic is FP64 with a fixed expression order; this file is
// compiled with -ffp-contract=off.
#include <stddef.h>

#include "internal.h"

namespace {

enum { SP_K0, SP_K1, SP_V0, SP_V1, SP_HIST, SP_N, SP_RS, SP_RE, SP_PROP, SP_UF, SP_RCI, SP_GRP, SP_KEPT, SP_NKEPT,
       SP_CAMS, SP_REM, SP_REMSCAN, SP_SCAN, SP_TOT, SP_COUNT };

constexpr double C0_SH = 0.28209479177387814;   // degree-0 real SH constant 1/(2 sqrt(pi))

struct Prop {
    double mu[3], R[9], s[3], rgb[3], Sig[9], Sinv[9];
    int32_t ok, view;
};

struct Group {
    double mu[3], R[9], s[3], rgb[3], extent;
};

__device__ __forceinline__ int64_t find_cand(const int32_t *cand, int64_t n_cand, int32_t id) {
    int64_t lo = 0, hi = n_cand;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (cand[mid] < id) lo = mid + 1;
        else hi = mid;
    }
    return (lo < n_cand && cand[lo] == id) ? lo : -1;
}

struct Parent {
    double mu[3], s[3], R[9], o;
};

__device__ __forceinline__ void load_parent(const GaussPtrs &g, int64_t i, Parent &p) {
    const int64_t n = g.n;
    for (int k = 0; k < 3; k++) p.mu[k] = (double)g.means[k * n + i];
    for (int k = 0; k < 3; k++) p.s[k] = exp((double)g.log_scales[k * n + i]);
    double q[4];
    for (int k = 0; k < 4; k++) q[k] = (double)g.quats[k * n + i];
    const double qnorm = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double w = q[0] / qnorm, x = q[1] / qnorm, y = q[2] / qnorm, z = q[3] / qnorm;
    p.R[0] = 1.0 - 2.0 * (y * y + z * z); p.R[1] = 2.0 * (x * y - w * z);       p.R[2] = 2.0 * (x * z + w * y);
    p.R[3] = 2.0 * (x * y + w * z);       p.R[4] = 1.0 - 2.0 * (x * x + z * z); p.R[5] = 2.0 * (y * z - w * x);
    p.R[6] = 2.0 * (x * z - w * y);       p.R[7] = 2.0 * (y * z + w * x);       p.R[8] = 1.0 - 2.0 * (x * x + y * y);
    p.o = 1.0 / (1.0 + exp(-(double)g.opac[i]));
}

__device__ __forceinline__ double clipv(double x, double a) {
    const double m = fabs(x) < a ? fabs(x) : a;
    return x < 0.0 ? -m : m;
}

// Child proposal of one region (App. A).
__device__ void make_proposal(const Parent &par, const as_region &r, const DevCam &cam, double eps, Prop &p) {
    p.ok = 0;
    double Rc[9], tc[3];
    for (int k = 0; k < 9; k++) Rc[k] = (double)cam.R[k];
    for (int k = 0; k < 3; k++) tc[k] = (double)cam.t[k];
    double ov[3];
    for (int j = 0; j < 3; j++) ov[j] = -(Rc[0 * 3 + j] * tc[0] + Rc[1 * 3 + j] * tc[1] + Rc[2 * 3 + j] * tc[2]);
    const double fx = cam.fx, fy = cam.fy;
    const double dc[3] = {(r.cx - (double)cam.cx) / fx, (r.cy - (double)cam.cy) / fy, 1.0};
    double dw[3];
    for (int j = 0; j < 3; j++) dw[j] = Rc[0 * 3 + j] * dc[0] + Rc[1 * 3 + j] * dc[1] + Rc[2 * 3 + j] * dc[2];
    const double dwn = sqrt(dw[0] * dw[0] + dw[1] * dw[1] + dw[2] * dw[2]);
    const double d[3] = {dw[0] / dwn, dw[1] / dwn, dw[2] / dwn};
    double Am[9];
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            double acc = 0.0;
            for (int k = 0; k < 3; k++) acc += par.R[a * 3 + k] * (1.0 / (par.s[k] * par.s[k])) * par.R[b * 3 + k];
            Am[a * 3 + b] = acc;
        }
    const double bv[3] = {par.mu[0] - ov[0], par.mu[1] - ov[1], par.mu[2] - ov[2]};
    double Ad[3];
    for (int a = 0; a < 3; a++) Ad[a] = Am[a * 3 + 0] * d[0] + Am[a * 3 + 1] * d[1] + Am[a * 3 + 2] * d[2];
    const double num = bv[0] * Ad[0] + bv[1] * Ad[1] + bv[2] * Ad[2];
    const double den = d[0] * Ad[0] + d[1] * Ad[1] + d[2] * Ad[2];
    const double tstar = num / (den + eps);
    for (int a = 0; a < 3; a++) p.mu[a] = ov[a] + tstar * d[a];
    const double dcn = sqrt(dc[0] * dc[0] + dc[1] * dc[1] + dc[2] * dc[2]);
    const double tz = tstar / dcn;
    if (!(tz > AS_NEAR)) return;
    double smax = par.s[0];
    if (par.s[1] > smax) smax = par.s[1];
    if (par.s[2] > smax) smax = par.s[2];
    const double e1x = r.e1[0], e1y = r.e1[1];
    const double e2x = -e1y, e2y = e1x;
    const double w1x = clipv(e1x * r.sigma1 * tz / fx, smax * fabs(e1x));
    const double w1y = clipv(e1y * r.sigma1 * tz / fy, smax * fabs(e1y));
    const double w2x = clipv(e2x * r.sigma2 * tz / fx, smax * fabs(e2x));
    const double w2y = clipv(e2y * r.sigma2 * tz / fy, smax * fabs(e2y));
    double a1[3], a2[3];
    for (int k = 0; k < 3; k++) {
        a1[k] = w1x * Rc[0 * 3 + k] + w1y * Rc[1 * 3 + k];
        a2[k] = w2x * Rc[0 * 3 + k] + w2y * Rc[1 * 3 + k];
    }
    const double n1 = sqrt(a1[0] * a1[0] + a1[1] * a1[1] + a1[2] * a1[2]);
    const double n2 = sqrt(a2[0] * a2[0] + a2[1] * a2[1] + a2[2] * a2[2]);
    if (!(n1 > 0.0) || !(n2 > 0.0)) return;
    p.s[0] = n1; p.s[1] = n2; p.s[2] = n2;
    const double u1[3] = {a1[0] / n1, a1[1] / n1, a1[2] / n1};
    const double pr = a2[0] * u1[0] + a2[1] * u1[1] + a2[2] * u1[2];
    const double q2[3] = {a2[0] - pr * u1[0], a2[1] - pr * u1[1], a2[2] - pr * u1[2]};
    const double nq = sqrt(q2[0] * q2[0] + q2[1] * q2[1] + q2[2] * q2[2]);
    if (!(nq > 0.0)) return;
    const double u2[3] = {q2[0] / nq, q2[1] / nq, q2[2] / nq};
    for (int k = 0; k < 3; k++) {
        p.R[k * 3 + 0] = u1[k];
        p.R[k * 3 + 1] = u2[k];
        p.R[k * 3 + 2] = Rc[2 * 3 + k];
    }
    for (int ch = 0; ch < 3; ch++) p.rgb[ch] = (double)r.rgb[ch];
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            double acc = 0.0, acci = 0.0;
            for (int k = 0; k < 3; k++) {
                acc += p.R[a * 3 + k] * (p.s[k] * p.s[k]) * p.R[b * 3 + k];
                acci += p.R[a * 3 + k] * (1.0 / (p.s[k] * p.s[k])) * p.R[b * 3 + k];
            }
            p.Sig[a * 3 + b] = acc;
            p.Sinv[a * 3 + b] = acci;
        }
    p.ok = 1;
}

__device__ __forceinline__ double maha(const double *Sinv, const double *dl) {
    double acc = 0.0;
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) acc += dl[a] * Sinv[a * 3 + b] * dl[b];
    return sqrt(acc);
}

// Cyclic Jacobi on a symmetric 3x3 matrix; columns of V are eigenvectors,
// sorted by descending eigenvalue, last column flipped so det V = +1.
__device__ void jacobi3(const double *Ain, double V[9], double lam[3]) {
    double A[9];
    for (int k = 0; k < 9; k++) A[k] = Ain[k];
    for (int k = 0; k < 9; k++) V[k] = (k % 4 == 0) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 32; sweep++) {
        const double off = A[1] * A[1] + A[2] * A[2] + A[5] * A[5];
        const double dia = A[0] * A[0] + A[4] * A[4] + A[8] * A[8];
        if (off <= 1e-30 * dia) break;
        for (int p = 0; p < 2; p++)
            for (int q = p + 1; q < 3; q++) {
                const double apq = A[p * 3 + q];
                if (apq == 0.0) continue;
                const double app = A[p * 3 + p], aqq = A[q * 3 + q];
                const double theta = (aqq - app) / (2.0 * apq);
                const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
                for (int k = 0; k < 3; k++) {
                    const double akp = A[k * 3 + p], akq = A[k * 3 + q];
                    A[k * 3 + p] = cs * akp - sn * akq;
                    A[k * 3 + q] = sn * akp + cs * akq;
                }
                for (int k = 0; k < 3; k++) {
                    const double apk = A[p * 3 + k], aqk = A[q * 3 + k];
                    A[p * 3 + k] = cs * apk - sn * aqk;
                    A[q * 3 + k] = sn * apk + cs * aqk;
                }
                for (int k = 0; k < 3; k++) {
                    const double vkp = V[k * 3 + p], vkq = V[k * 3 + q];
                    V[k * 3 + p] = cs * vkp - sn * vkq;
                    V[k * 3 + q] = sn * vkp + cs * vkq;
                }
            }
    }
    for (int k = 0; k < 3; k++) lam[k] = A[k * 4];
    for (int a = 0; a < 2; a++) {
        int best = a;
        for (int b = a + 1; b < 3; b++)
            if (lam[b] > lam[best]) best = b;
        if (best != a) {
            const double tl = lam[a];
            lam[a] = lam[best];
            lam[best] = tl;
            for (int k = 0; k < 3; k++) {
                const double tv = V[k * 3 + a];
                V[k * 3 + a] = V[k * 3 + best];
                V[k * 3 + best] = tv;
            }
        }
    }
    const double det = V[0] * (V[4] * V[8] - V[5] * V[7]) - V[1] * (V[3] * V[8] - V[5] * V[6]) +
                       V[2] * (V[3] * V[7] - V[4] * V[6]);
    if (det < 0.0)
        for (int k = 0; k < 3; k++) V[k * 3 + 2] = -V[k * 3 + 2];
}

// Unit quaternion (w >= 0) of a rotation matrix (Shepperd's method).
__device__ void rot_to_quat(const double *R, double q[4]) {
    const double tr = R[0] + R[4] + R[8];
    double w, x, y, z;
    if (tr > 0.0) {
        const double s = sqrt(tr + 1.0) * 2.0;
        w = 0.25 * s; x = (R[7] - R[5]) / s; y = (R[2] - R[6]) / s; z = (R[3] - R[1]) / s;
    } else if (R[0] > R[4] && R[0] > R[8]) {
        const double s = sqrt(1.0 + R[0] - R[4] - R[8]) * 2.0;
        w = (R[7] - R[5]) / s; x = 0.25 * s; y = (R[1] + R[3]) / s; z = (R[2] + R[6]) / s;
    } else if (R[4] > R[8]) {
        const double s = sqrt(1.0 + R[4] - R[0] - R[8]) * 2.0;
        w = (R[2] - R[6]) / s; x = (R[1] + R[3]) / s; y = 0.25 * s; z = (R[5] + R[7]) / s;
    } else {
        const double s = sqrt(1.0 + R[8] - R[0] - R[4]) * 2.0;
        w = (R[3] - R[1]) / s; x = (R[2] + R[6]) / s; y = (R[5] + R[7]) / s; z = 0.25 * s;
    }
    double nn = sqrt(w * w + x * x + y * y + z * z);
    if (w < 0.0) nn = -nn;
    q[0] = w / nn; q[1] = x / nn; q[2] = y / nn; q[3] = z / nn;
}

// ---- kernels ----------------------------------------------------------------------------

__global__ void k_reg_prep(const int64_t *__restrict__ count, int64_t cap, uint32_t *__restrict__ n32) {
    const int64_t c = *count;
    *n32 = (uint32_t)(c < cap ? c : cap);
}

__global__ void k_reg_keys(const as_region *__restrict__ recs, const uint32_t *__restrict__ n32, int64_t cap, int lb,
                           int vb, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cap || i >= (int64_t)*n32) return;
    const as_region &r = recs[i];
    keys[i] = ((uint64_t)(uint32_t)r.cand << (vb + lb)) | ((uint64_t)(uint32_t)r.view << lb) | (uint64_t)(uint32_t)r.label;
    vals[i] = (uint32_t)i;
}

// Region waves: kernels over the sorted regions take a bounded grid and stride,
// because the region capacity the host knows is far above the regions in use
// (a grid over the capacity launched 6,500 blocks for 6,400 regions).
constexpr int RW_BLOCKS = 2048;

// Zeroes what the split accumulates into: the candidates' region ranges and
// root counts, and the removal mask (one launch instead of three fills).
__global__ void k_split_init(int64_t nc, int64_t n, int64_t *__restrict__ rs, int64_t *__restrict__ re,
                             int32_t *__restrict__ nkept, uint8_t *__restrict__ removed) {
    const int64_t st = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nc || i < n; i += st) {
        if (i < nc) {
            rs[i] = 0;
            re[i] = 0;
            nkept[i] = 0;
        }
        if (i < n) removed[i] = 0;
    }
}

// One thread per sorted region: its candidate (rci, -1 if none), the
// candidate's region range, its child proposal and its union-find cell (the
// region itself, or -1 without a proposal).
__global__ void __launch_bounds__(256) k_propose(GaussPtrs g, const as_region *__restrict__ recs,
                                                 const uint32_t *__restrict__ order, const uint32_t *__restrict__ n32,
                                                 int64_t cap, const int32_t *__restrict__ cand, int64_t n_cand,
                                                 const int64_t *__restrict__ n_cand_dev,
                                                 const DevCam *__restrict__ cams, int n_views, double eps,
                                                 int64_t *__restrict__ rs, int64_t *__restrict__ re,
                                                 int32_t *__restrict__ rci, int32_t *__restrict__ uf,
                                                 Prop *__restrict__ props) {
    const int64_t R = (int64_t)*n32 < cap ? (int64_t)*n32 : cap;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < R; i += (int64_t)gridDim.x * blockDim.x) {
        const as_region r = recs[order[i]];
        Prop p;
        p.ok = 0;
        p.view = r.view;
        const int64_t ci = find_cand(cand, count_in_use(n_cand, n_cand_dev), r.cand);
        if (ci >= 0) {
            if (i == 0 || recs[order[i - 1]].cand != r.cand) rs[ci] = i;
            if (i == R - 1 || recs[order[i + 1]].cand != r.cand) re[ci] = i + 1;
            if (r.view >= 0 && r.view < n_views && r.cand < rows_in_use(g)) {
                Parent par;
                load_parent(g, r.cand, par);
                make_proposal(par, r, cams[r.view], eps, p);
            }
        }
        rci[i] = (int32_t)ci;
        uf[i] = p.ok ? (int32_t)i : -1;
        props[i] = p;
    }
}

__device__ __forceinline__ int32_t uf_load(const int32_t *L, int64_t x) {
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

// The merge of Eq. (merge_conditions) and Eq. (merge_cov) runs with one wave per
// region, not per candidate: the candidates are very uneven (most hold none
// or a few regions, one held several hundred of the 6,400 regions of 16 views over 500,000
// Gaussians), so a wave per candidate left the chip waiting on one wave that
// took every pair test, group sum and rank of its candidate in sequence
// (1572 us there; see k_rank for the time now).  Three launches, because
// each needs the whole candidate of the one before.

// Eq. (merge_conditions): the wave of region a tests it against the later
// regions of its candidate, a lane each, and unites those that merge.
__global__ void __launch_bounds__(256) k_pairs(const uint32_t *__restrict__ n32, int64_t cap,
                                               const int32_t *__restrict__ rci, const int64_t *__restrict__ re_a,
                                               const Prop *__restrict__ props, int32_t *uf, double gamma_d,
                                               double gamma_c, uint32_t flags) {
    const int lane = threadIdx.x & 63;
    const int64_t R = (int64_t)*n32 < cap ? (int64_t)*n32 : cap;
    for (int64_t a = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); a < R; a += (int64_t)gridDim.x * 4) {
        const int32_t ci = rci[a];
        if (ci < 0 || !props[a].ok) continue;
        const Prop &pa = props[a];
        const int64_t re = re_a[ci];
        for (int64_t b = a + 1 + lane; b < re; b += 64) {
            const Prop &pb = props[b];
            if (!pb.ok) continue;
            if ((flags & AS_SPLIT_CROSS_VIEW) && pb.view == pa.view) continue;
            const double dl[3] = {pb.mu[0] - pa.mu[0], pb.mu[1] - pa.mu[1], pb.mu[2] - pa.mu[2]};
            const double dm = maha(pa.Sinv, dl) + maha(pb.Sinv, dl);
            double dc = 0.0;
            for (int ch = 0; ch < 3; ch++) {
                const double t = fabs(pa.rgb[ch] - pb.rgb[ch]);
                if (t > dc) dc = t;
            }
            if (dm <= gamma_d && dc <= gamma_c) uf_unite(uf, (int32_t)a, (int32_t)b);
        }
    }
}

// Eq. (merge_cov): one merged child per group, at the group's first member.
// The wave finds the members by ballots over the candidate's later regions;
// lane k < 15 sums component k of the members' means, colours and covariances
// in member order (the sums keep their order, only the components run side by
// side), four members' loads in flight, and the extents' maxima take a lane per member.
__global__ void __launch_bounds__(256) k_groups(const uint32_t *__restrict__ n32, int64_t cap,
                                                const int32_t *__restrict__ rci, const int64_t *__restrict__ re_a,
                                                const Prop *__restrict__ props, const int32_t *__restrict__ uf,
                                                uint32_t flags, Group *__restrict__ grp) {
    const int lane = threadIdx.x & 63;
    const int64_t R = (int64_t)*n32 < cap ? (int64_t)*n32 : cap;
    // offset of component `lane` in Prop (doubles): mu, then rgb and Sig
    static_assert(offsetof(Prop, rgb) == 15 * 8 && offsetof(Prop, Sig) == 18 * 8, "component offsets");
    const int comp = lane < 3 ? lane : 12 + (lane < 15 ? lane : 3);
    for (int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); j < R; j += (int64_t)gridDim.x * 4) {
        const int32_t ci = rci[j];
        if (ci < 0 || uf[j] != (int32_t)j) continue;   // wave-uniform
        const int64_t re = re_a[ci];
        double acc = 0.0;
        int64_t M = 0;
        for (int64_t m0 = j; m0 < re; m0 += 64) {
            const int64_t m = m0 + lane;
            uint64_t in = __ballot(m < re && uf[m] >= 0 && uf_find(uf, (int32_t)m) == (int32_t)j);
            M += __popcll(in);
            while (in) {
                double x[4];
                int k = 0;
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (in) {
                        const int b = __ffsll((unsigned long long)in) - 1;
                        in &= in - 1;
                        x[u] = reinterpret_cast<const double *>(props + m0 + b)[comp];
                        k = u + 1;
                    }
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (u < k) acc += x[u];
            }
        }
        Group gr;
        if (M == 1) {
            const Prop &pj = props[j];
            for (int k = 0; k < 3; k++) { gr.mu[k] = pj.mu[k]; gr.rgb[k] = pj.rgb[k]; gr.s[k] = pj.s[k]; }
            for (int k = 0; k < 9; k++) gr.R[k] = pj.R[k];
        } else {
            const double mean = acc / (double)M;
            double Sbar[9];
            for (int k = 0; k < 3; k++) { gr.mu[k] = __shfl(mean, k, 64); gr.rgb[k] = __shfl(mean, 3 + k, 64); }
            for (int k = 0; k < 9; k++) Sbar[k] = __shfl(mean, 6 + k, 64);
            double E[9], lam[3];
            jacobi3(Sbar, E, lam);
            double best[3] = {0.0, 0.0, 0.0};
            for (int64_t m = j + lane; m < re; m += 64) {
                if (uf[m] < 0 || uf_find(uf, (int32_t)m) != (int32_t)j) continue;
                const Prop &pm = props[m];
                for (int r = 0; r < 3; r++) {
                    const double er[3] = {E[0 * 3 + r], E[1 * 3 + r], E[2 * 3 + r]};
                    const double off = fabs(er[0] * (pm.mu[0] - gr.mu[0]) + er[1] * (pm.mu[1] - gr.mu[1]) +
                                            er[2] * (pm.mu[2] - gr.mu[2]));
                    double Se[3];
                    for (int k = 0; k < 3; k++)
                        Se[k] = pm.Sig[k * 3 + 0] * er[0] + pm.Sig[k * 3 + 1] * er[1] + pm.Sig[k * 3 + 2] * er[2];
                    const double sig = sqrt(er[0] * Se[0] + er[1] * Se[1] + er[2] * Se[2]);
                    const double reach = off + sig;
                    if (reach > best[r]) best[r] = reach;
                }
            }
            for (int r = 0; r < 3; r++) {
                for (int o = 32; o > 0; o >>= 1) {
                    const double t = __shfl_xor(best[r], o, 64);
                    if (t > best[r]) best[r] = t;
                }
                gr.s[r] = best[r];
            }
            for (int k = 0; k < 9; k++) gr.R[k] = E[k];
        }
        if (flags & AS_SPLIT_EXTENT_MAX) {
            double m = gr.s[0];
            if (gr.s[1] > m) m = gr.s[1];
            if (gr.s[2] > m) m = gr.s[2];
            gr.extent = m;
        } else {
            gr.extent = gr.s[0] * gr.s[1] * gr.s[2];
        }
        if (lane == 0) grp[j] = gr;
    }
}

// An extent as it is ranked (a proposal of non-finite parameters ranks last).
__device__ __forceinline__ double rank_extent(double e) { return e == e ? e : -1.0; }

// A group's rank among its candidate's by (extent descending, first member
// ascending): the wave of its root counts the groups ahead of it.  The first
// n_max are kept; nroots counts the candidate's groups.
// Merge, groups, ranks and modes together, 16 views over 500,000 Gaussians with
// 25,167 candidates and 6,374 regions: 31 us (7 + 16 + 4 + 4).
__global__ void __launch_bounds__(256) k_rank(const uint32_t *__restrict__ n32, int64_t cap,
                                              const int32_t *__restrict__ rci, const int64_t *__restrict__ rs_a,
                                              const int64_t *__restrict__ re_a, const int32_t *__restrict__ uf,
                                              const Group *__restrict__ grp, int n_max, int32_t *__restrict__ kept,
                                              int32_t *__restrict__ nroots) {
    const int lane = threadIdx.x & 63;
    const int64_t R = (int64_t)*n32 < cap ? (int64_t)*n32 : cap;
    for (int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); j < R; j += (int64_t)gridDim.x * 4) {
        const int32_t ci = rci[j];
        if (ci < 0 || uf[j] != (int32_t)j) continue;   // wave-uniform
        const int64_t rs = rs_a[ci], re = re_a[ci];
        const double ej = rank_extent(grp[j].extent);
        int32_t rank = 0;
        for (int64_t h = rs + lane; h < re; h += 64) {
            if (h == j || uf[h] != (int32_t)h) continue;
            const double eh = rank_extent(grp[h].extent);
            if (eh > ej || (eh == ej && h < j)) rank++;
        }
        for (int o = 32; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 64);
        if (lane == 0) {
            if (rank < n_max) kept[rs + rank] = (int32_t)j;
            atomicAdd(nroots + ci, 1);
        }
    }
}

// One thread per candidate: its mode, its row count, the groups it keeps
// (nkept holds the groups found on entry) and whether its parent leaves.
__global__ void __launch_bounds__(256) k_modes(const int32_t *__restrict__ cand, int64_t n_cand,
                                               const int64_t *__restrict__ n_cand_dev,
                                               const int32_t *__restrict__ attr, int n_max, int variant, int fixed_n,
                                               int32_t *__restrict__ nkept, uint8_t *__restrict__ mode,
                                               int32_t *__restrict__ count, uint8_t *__restrict__ removed) {
    const int64_t ci = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ci >= n_cand) return;
    uint8_t md = 0;
    int32_t cnt = 0, nk = 0;
    if (ci < count_in_use(n_cand, n_cand_dev)) {   // capacity past the candidates in use: no rows
        const int32_t id = cand[ci];
        nk = nkept[ci] < n_max ? nkept[ci] : n_max;
        if (variant == AS_VARIANT_FIXED_N) { md = 3; cnt = fixed_n; nk = 0; }   // whatever the regions say
        else if (attr[id] == 0) { md = 0; cnt = 2; }
        else if (nk == 0) { md = 1; cnt = 0; }
        else if (variant == AS_VARIANT_ADAPTIVE_N) { md = 3; cnt = nk; }   // as many random children as proposals
        else { md = 2; cnt = nk + 1; }
        if (md != 1) removed[id] = 1;
    }
    mode[ci] = md;
    count[ci] = cnt;
    nkept[ci] = nk;
}

// A set's parameter rows in chunks of at most 12: chunk 0 is the geometry
// (means, log scales, quaternion, opacity), the rest SH rows.  A thread loads
// a chunk before it stores any of it: loads and stores of sets that may
// alias are otherwise kept in order, a memory latency per row.
constexpr int ROW_CHUNK = 12;
__host__ __device__ __forceinline__ int row_chunks(int deg) {
    return 1 + (3 * (deg + 1) * (deg + 1) + ROW_CHUNK - 1) / ROW_CHUNK;
}
// Rows of chunk c of a Gaussian, and their place in an output set.
__device__ __forceinline__ int chunk_rows(int c, int deg) {
    if (c == 0) return 11;
    const int left = 3 * (deg + 1) * (deg + 1) - ROW_CHUNK * (c - 1);
    return left < ROW_CHUNK ? left : ROW_CHUNK;
}
__device__ __forceinline__ void load_chunk(const GaussPtrs &g, int64_t i, int c, int rows, float v[ROW_CHUNK]) {
    const int64_t n = g.n;
    if (c == 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) v[k] = g.means[k * n + i];
#pragma unroll
        for (int k = 0; k < 3; k++) v[3 + k] = g.log_scales[k * n + i];
#pragma unroll
        for (int k = 0; k < 4; k++) v[6 + k] = g.quats[k * n + i];
        v[10] = g.opac[i];
        return;
    }
    const float *sh = g.sh + (int64_t)ROW_CHUNK * (c - 1) * n;
#pragma unroll
    for (int k = 0; k < ROW_CHUNK; k++)
        if (k < rows) v[k] = sh[k * n + i];
}
__device__ __forceinline__ void store_chunk(const GradPtrs &o, int64_t i, int c, int rows, const float v[ROW_CHUNK]) {
    const int64_t n = o.stride;
    if (c == 0) {
#pragma unroll
        for (int k = 0; k < 3; k++) o.means[k * n + i] = v[k];
#pragma unroll
        for (int k = 0; k < 3; k++) o.log_scales[k * n + i] = v[3 + k];
#pragma unroll
        for (int k = 0; k < 4; k++) o.quats[k * n + i] = v[6 + k];
        o.opac[i] = v[10];
        return;
    }
    float *sh = o.sh + (int64_t)ROW_CHUNK * (c - 1) * n;
#pragma unroll
    for (int k = 0; k < ROW_CHUNK; k++)
        if (k < rows) sh[k * n + i] = v[k];
}

// grid.y: chunk of rows
__global__ void __launch_bounds__(256) k_copy_survivors(GaussPtrs g, const uint8_t *__restrict__ removed,
                                                        const int64_t *__restrict__ rem_prefix, GradPtrs out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows_in_use(g) || removed[i]) return;
    const int c = blockIdx.y, rows = chunk_rows(c, g.deg);
    float v[ROW_CHUNK];
    load_chunk(g, i, c, rows, v);
    store_chunk(out, i - rem_prefix[i], c, rows, v);
}

// A thread per (candidate, chunk of rows, residue of the child index modulo
// CHILD_LANES).  With one thread per candidate writing all rows of all its
// children the kernel took 127 us for 25,167 candidates of SH degree 3 (each
// row a dependent load and store); with the rows chunked 54 us, the time of the
// candidates of 20 children (two square roots, a division and three
// logarithms each); 36 us with those spread over lanes as well.
constexpr int CHILD_LANES = 8;
__global__ void __launch_bounds__(64) k_write_children(GaussPtrs g, const int32_t *__restrict__ cand, int64_t n_cand,
                                                       const int64_t *__restrict__ n_cand_dev,
                                                       const uint8_t *__restrict__ mode,
                                                       const int64_t *__restrict__ offset,
                                                       const int64_t *__restrict__ tot,
                                                       const int64_t *__restrict__ rs_a,
                                                       const Group *__restrict__ grp_all,
                                                       const int32_t *__restrict__ kept_all,
                                                       const int32_t *__restrict__ count,
                                                       const float *__restrict__ noise, int noise_n, double eta,
                                                       uint32_t flags, GradPtrs out, int64_t *__restrict__ n_out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, ci = t / CHILD_LANES;
    const int c = blockIdx.y;
    const int64_t n_surv = rows_in_use(g) - tot[0];
    if (t == 0 && c == 0) *n_out = n_surv + tot[1];
    if (ci >= count_in_use(n_cand, n_cand_dev)) return;
    const uint8_t md = mode[ci];
    const int32_t N = count[ci], r0 = (int32_t)(t % CHILD_LANES);
    if (md == 1 || r0 >= N) return;
    const int64_t base = n_surv + offset[ci];
    const int32_t id = cand[ci];
    const int rows = chunk_rows(c, g.deg);
    float v[ROW_CHUNK];   // the parent's rows
    load_chunk(g, id, c, rows, v);
    if (md == 0 || md == 3) {
        // Eq. (vanilla_split_sample), Eq. (vanilla_split_scale) with N = count
        // (2 for the VANILLA fallback)
        if (c > 0) {
            for (int32_t r = r0; r < N; r += CHILD_LANES) store_chunk(out, base + r, c, rows, v);
            return;
        }
        Parent par;
        load_parent(g, id, par);
        const double shrink = log(eta * (double)N);
        for (int k = 0; k < 3; k++) v[3 + k] = (float)((double)v[3 + k] - shrink);
        for (int32_t r = r0; r < N; r += CHILD_LANES) {
            double dl[3];
            for (int k = 0; k < 3; k++) dl[k] = par.s[k] * (double)noise[((int64_t)ci * noise_n + r) * 3 + k];
            for (int k = 0; k < 3; k++)
                v[k] = (float)(par.mu[k] + (par.R[k * 3 + 0] * dl[0] + par.R[k * 3 + 1] * dl[1] + par.R[k * 3 + 2] * dl[2]));
            store_chunk(out, base + r, 0, 11, v);
        }
        return;
    }
    // the kept groups (N - 1 of them), then the parent's copy
    const int64_t rs = rs_a[ci];
    const int32_t ng = N - 1;
    const double o = 1.0 / (1.0 + exp(-(double)v[10]));   // chunk 0 only
    const double pr = o / (double)(ng + 1);
    const float shared = (float)log(pr / (1.0 - pr));
    for (int32_t r = r0; r < N; r += CHILD_LANES) {
        if (r == ng) {
            if (c == 0) v[10] = shared;
            store_chunk(out, base + r, c, rows, v);
            break;
        }
        float w[ROW_CHUNK];
        for (int k = 0; k < ROW_CHUNK; k++) w[k] = 0.0f;
        if (c <= 1) {
            const Group &gr = grp_all[kept_all[rs + r]];
            if (c == 1) {
                for (int ch = 0; ch < 3; ch++) w[ch] = (float)((gr.rgb[ch] - 0.5) / C0_SH);
            } else {
                double q[4];
                rot_to_quat(gr.R, q);
                for (int k = 0; k < 3; k++) w[k] = (float)gr.mu[k];
                for (int k = 0; k < 3; k++) w[3 + k] = (float)log(gr.s[k]);
                for (int k = 0; k < 4; k++) w[6 + k] = (float)q[k];
                // Eq. (child_params): the parent's opacity (second reading: every row of the block at o/(N+1))
                w[10] = (flags & AS_SPLIT_SHARE_OPACITY) ? shared : v[10];
            }
        }
        store_chunk(out, base + r, c, rows, w);
    }
}

int bits_for(int64_t v) {   // bits needed to represent 0..v
    int b = 1;
    while ((int64_t(1) << b) <= v && b < 62) b++;
    return b;
}

constexpr int CAM_CHUNK = 16;
struct CamChunk {
    int m;
    DevCam cam[CAM_CHUNK];
};
__global__ void k_store_cams(const CamChunk c, DevCam *__restrict__ dst) {
    if ((int)threadIdx.x < c.m) dst[threadIdx.x] = c.cam[threadIdx.x];
}

}  // namespace

// Bytes of each scratch slot for region capacity `cap`, `nc` candidates, `nv`
// views and `n` Gaussians: the region sort's keys, values and histogram, the
// candidates' region ranges, proposals, union-find, groups and kept lists,
// the camera table, the removal mask and its scan.
static void sp_need(int64_t cap, int64_t nc, int64_t nv, int64_t n, size_t need[SP_COUNT]) {
    cap = cap > 0 ? cap : 1;
    nc = nc > 0 ? nc : 1;
    nv = nv > 0 ? nv : 1;
    n = n > 0 ? n : 1;
    const size_t v[SP_COUNT] = {(size_t)cap * 8, (size_t)cap * 8, (size_t)cap * 4, (size_t)cap * 4, sort_hist_bytes(cap),
                                64, (size_t)nc * 8, (size_t)nc * 8, (size_t)cap * sizeof(Prop), (size_t)cap * 4,
                                (size_t)cap * 4, (size_t)cap * sizeof(Group), (size_t)cap * 4, (size_t)nc * 4,
                                (size_t)nv * sizeof(DevCam), (size_t)n, (size_t)n * 8, scan_tmp_bytes(n > nc ? n : nc),
                                64};
    for (int k = 0; k < SP_COUNT; k++) need[k] = v[k];
}

size_t split_reserve_bytes(const as_reserve &r) {
    size_t need[SP_COUNT], total = 0;
    sp_need(r.max_regions, r.max_candidates, r.max_views, r.max_gaussians, need);
    for (int k = 0; k < SP_COUNT; k++) total += devbuf_size(need[k]);
    return total;
}

hipError_t split_reserve(as_ctx *ctx, const as_reserve &r) {
    size_t need[SP_COUNT];
    sp_need(r.max_regions, r.max_candidates, r.max_views, r.max_gaussians, need);
    hipError_t e = hipSuccess;
    for (int k = 0; k < SP_COUNT && e == hipSuccess; k++) e = devbuf_ensure(ctx->sp[k], need[k]);
    return e;
}

as_status run_adaptive_split(as_ctx *ctx, const GaussPtrs &g, const int32_t *cand, int64_t n_cand,
                             const int64_t *n_cand_dev, const as_region_buf &rb, const as_camera *views, int n_views, const int32_t *attr,
                             const as_split_params &p, const float *noise, GradPtrs out, int64_t out_cap,
                             uint8_t *mode, int32_t *count, int64_t *offset, int64_t *n_out, hipStream_t s) {
    (void)out_cap;
    const int64_t cap = rb.capacity > 0 ? rb.capacity : 1;
    int64_t max_px = 1;
    for (int v = 0; v < n_views; v++) {
        const int64_t px = (int64_t)views[v].width * views[v].height;
        if (px > max_px) max_px = px;
    }
    const int lb = bits_for(max_px), vb = bits_for(n_views > 0 ? n_views : 1), cb = bits_for(g.n);
    if (lb + vb + cb > 64) {
        as_set_error("region sort key needs %d bits (> 64)", lb + vb + cb);
        return AS_ERR_ARG;
    }
    // the scratch sizes of sp_need (every count at least 1) must be reserved
    const int64_t nc1 = n_cand > 0 ? n_cand : 1, nv1 = n_views > 0 ? n_views : 1, n1 = g.n > 0 ? g.n : 1;
    const as_reserve &res = ctx->res;
    if (cap > res.max_regions || nc1 > res.max_candidates || nv1 > res.max_views || n1 > res.max_gaussians) {
        as_set_error("as_adaptive_split: needs max_regions >= %lld, max_candidates >= %lld, max_views >= %lld, "
                     "max_gaussians >= %lld in as_ctx_reserve (reserved %lld, %lld, %d, %lld)", (long long)cap,
                     (long long)nc1, (long long)nv1, (long long)n1, (long long)res.max_regions,
                     (long long)res.max_candidates, res.max_views, (long long)res.max_gaussians);
        return AS_ERR_CAPACITY;
    }
    DevBuf *sp = ctx->sp;
    uint64_t *keys[2] = {(uint64_t *)sp[SP_K0].p, (uint64_t *)sp[SP_K1].p};
    uint32_t *vals[2] = {(uint32_t *)sp[SP_V0].p, (uint32_t *)sp[SP_V1].p};
    uint32_t *n32 = (uint32_t *)sp[SP_N].p;
    int64_t *rs = (int64_t *)sp[SP_RS].p, *re = (int64_t *)sp[SP_RE].p, *tot = (int64_t *)sp[SP_TOT].p;
    Prop *props = (Prop *)sp[SP_PROP].p;
    Group *grp = (Group *)sp[SP_GRP].p;
    int32_t *uf = (int32_t *)sp[SP_UF].p, *rci = (int32_t *)sp[SP_RCI].p, *kept = (int32_t *)sp[SP_KEPT].p;
    int32_t *nkept = (int32_t *)sp[SP_NKEPT].p;
    DevCam *dcams = (DevCam *)sp[SP_CAMS].p;
    uint8_t *removed = (uint8_t *)sp[SP_REM].p;
    int64_t *remscan = (int64_t *)sp[SP_REMSCAN].p;

    // cameras travel as kernel arguments (no host copy, no synchronisation)
    for (int v0 = 0; v0 < n_views; v0 += CAM_CHUNK) {
        CamChunk cc;
        cc.m = n_views - v0 < CAM_CHUNK ? n_views - v0 : CAM_CHUNK;
        for (int k = 0; k < cc.m; k++) cc.cam[k] = to_devcam(views[v0 + k]);
        hipLaunchKernelGGL(k_store_cams, dim3(1), dim3(64), 0, s, cc, dcams + v0);
    }
    const unsigned gcap = (unsigned)((cap + 255) / 256);
    const int64_t zn = nc1 > n1 ? nc1 : n1;
    hipLaunchKernelGGL(k_split_init, dim3((unsigned)(zn < 2048 * 256 ? (zn + 255) / 256 : 2048)), dim3(256), 0, s, nc1,
                       g.n, rs, re, nkept, removed);
    if (p.variant != AS_VARIANT_FIXED_N) {   // the fixed-N split reads no region
        hipLaunchKernelGGL(k_reg_prep, dim3(1), dim3(1), 0, s, rb.count, cap, n32);
        hipLaunchKernelGGL(k_reg_keys, dim3(gcap), dim3(256), 0, s, rb.records, n32, cap, lb, vb, keys[0], vals[0]);
        const int sel = radix_sort_u64(keys, vals, n32, cap, cap, 0, lb + vb + cb, 8, sp[SP_HIST].p, s);
        const uint32_t *order = vals[sel];
        const dim3 tg(gcap < RW_BLOCKS ? gcap : RW_BLOCKS), wg((unsigned)(cap < 4 * RW_BLOCKS ? (cap + 3) / 4 : RW_BLOCKS));
        hipLaunchKernelGGL(k_propose, tg, dim3(256), 0, s, g, rb.records, order, n32, cap, cand, n_cand, n_cand_dev,
                           dcams, n_views, p.eps, rs, re, rci, uf, props);
        if (n_cand > 0) {
            if (p.variant == AS_VARIANT_ADPSPLIT)   // the ablation variants do not merge
                hipLaunchKernelGGL(k_pairs, wg, dim3(256), 0, s, n32, cap, rci, re, props, uf, p.gamma_d, p.gamma_c,
                                   p.flags);
            hipLaunchKernelGGL(k_groups, wg, dim3(256), 0, s, n32, cap, rci, re, props, uf, p.flags, grp);
            hipLaunchKernelGGL(k_rank, wg, dim3(256), 0, s, n32, cap, rci, rs, re, uf, grp, p.n_max, kept, nkept);
        }
    }
    if (n_cand > 0)
        hipLaunchKernelGGL(k_modes, dim3((unsigned)((n_cand + 255) / 256)), dim3(256), 0, s, cand, n_cand, n_cand_dev,
                           attr, p.n_max, p.variant, p.fixed_n, nkept, mode, count, removed);
    scan_i32_to_i64(count, offset, n_cand, tot + 1, sp[SP_SCAN].p, s);
    scan_u8_to_i64(removed, remscan, g.n, tot, sp[SP_SCAN].p, s);
    if (g.n > 0)
        hipLaunchKernelGGL(k_copy_survivors, dim3((unsigned)((g.n + 255) / 256), row_chunks(g.deg)), dim3(256), 0, s, g,
                           removed, remscan, out);
    hipLaunchKernelGGL(k_write_children, dim3((unsigned)((CHILD_LANES * nc1 + 63) / 64), row_chunks(g.deg)), dim3(64), 0, s, g, cand,
                       n_cand, n_cand_dev, mode,
                       offset, tot, rs, grp, kept, count, noise, p.noise_n ? p.noise_n : 2, p.eta, p.flags, out,
                       n_out);
    return AS_OK;
}

AS_WARM_KERNEL(split)
