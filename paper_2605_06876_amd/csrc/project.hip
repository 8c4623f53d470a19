// EWA projection, spherical-harmonic colour, depth key and compact box of every
// Gaussian (Sec. 3 of the paper: each Gaussian is projected to the image plane
// and its view-dependent colour decoded from SH along the viewing direction).
//
// One thread per (view, Gaussian) entry, struct-of-arrays reads (coalesced), or
// per Gaussian of a set that several views show (k_project_views).  All arithmetic
// is FP64 and this file is compiled with -ffp-contract=off: the depth key and
// the pixel box decide which (tile, Gaussian) pairs exist, so they are
// computed with a fixed expression order and IEEE-rounded operations.
#include <string.h>

#include "internal.h"
#include "sh_device.h"

namespace {

__device__ __forceinline__ void quat_to_rot_d(double w, double x, double y, double z, double R[9]) {
    R[0] = 1.0 - 2.0 * (y * y + z * z); R[1] = 2.0 * (x * y - w * z);       R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);       R[4] = 1.0 - 2.0 * (x * x + z * z); R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);       R[7] = 2.0 * (y * z + w * x);       R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// What a Gaussian's projections into any view share: its centre, covariance,
// opacity and the box's exponent bound.
struct Shape {
    double mu[3], S[9], o, kk;
};

__device__ __forceinline__ Shape shape_of(const double mu[3], const double s[3], const double q[4], double ologit) {
    Shape sp;
    for (int k = 0; k < 3; k++) sp.mu[k] = mu[k];
    const double qn2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3];
    const double qnorm = sqrt(qn2);
    double Rg[9];
    quat_to_rot_d(q[0] / qnorm, q[1] / qnorm, q[2] / qnorm, q[3] / qnorm, Rg);
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            double acc = 0.0;
            for (int k = 0; k < 3; k++) acc += Rg[a * 3 + k] * (s[k] * s[k]) * Rg[b * 3 + k];
            sp.S[a * 3 + b] = acc;
        }
    sp.o = 1.0 / (1.0 + exp(-ologit));
    sp.kk = 2.0 * log(255.0 * sp.o);
    return sp;
}

template <int NK3, bool BUF>
__device__ __forceinline__ void load_sh(const GaussPtrs &g, uint32_t bo, float (&shv)[NK3]) {
    const int64_t n = g.n;
    if constexpr (BUF) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.sh), (short)0, -1,
                                                                            AS_BUFFER_RSRC_WORD3);
#pragma unroll
        for (int k = 0; k < NK3; k++)
            shv[k] = __uint_as_float(
                __builtin_amdgcn_raw_buffer_load_b32(r, (int)bo, (int)((uint32_t)k * (uint32_t)n * 4u), 0));
    } else {
#pragma unroll
        for (int k = 0; k < NK3; k++) shv[k] = at_row(g.sh, k, n, bo);
    }
}

// One entry in front of the camera: record, box and tile count (left alone
// when it is culled, apart from rec's colour, which is then zero).
template <int DEG>
__device__ __forceinline__ void project_entry(const Shape &sp, const float *shv, const DevCam &cam, const double Rc[9],
                                              const double tc[3], const double tv[3], int bs, BlendRec &rr, short4 &bx,
                                              uint32_t &nt) {
    constexpr int nk = (DEG + 1) * (DEG + 1);
    const double fx = cam.fx, fy = cam.fy, cx = cam.cx, cy = cam.cy;
    const double tx = tv[0], ty = tv[1], tz = tv[2];
    // perspective Jacobian at the (clamped) centre
    const double limx = 1.3 * ((double)cam.W / (2.0 * fx));
    const double limy = 1.3 * ((double)cam.H / (2.0 * fy));
    const double txtz = tx / tz, tytz = ty / tz;
    const double cx_ = fmin(limx, fmax(-limx, txtz)) * tz;
    const double cy_ = fmin(limy, fmax(-limy, tytz)) * tz;
    const double J[6] = {fx / tz, 0.0, -(fx * cx_) / (tz * tz), 0.0, fy / tz, -(fy * cy_) / (tz * tz)};
    double T[6];
    for (int r = 0; r < 2; r++)
        for (int k = 0; k < 3; k++)
            T[r * 3 + k] = J[r * 3 + 0] * Rc[0 * 3 + k] + J[r * 3 + 1] * Rc[1 * 3 + k] + J[r * 3 + 2] * Rc[2 * 3 + k];
    double C2[4];
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) {
            double acc = 0.0;
            for (int k = 0; k < 3; k++)
                for (int l = 0; l < 3; l++) acc += T[a * 3 + k] * sp.S[k * 3 + l] * T[b * 3 + l];
            C2[a * 2 + b] = acc;
        }
    const double A = C2[0] + AS_LOWPASS, B = C2[1], Cc = C2[3] + AS_LOWPASS;
    const double det = A * Cc - B * B;
    // The culling tests below are taken together after the colour, so
    // the code from the SH loads to the end is one block: the compiler
    // neither sinks the loads to their use nor splits the arithmetic
    // around them (a culled entry computes NaNs or values it discards).
    const double mx = fx * tx / tz + cx;
    const double my = fy * ty / tz + cy;
    const double hx = sqrt(sp.kk * A), hy = sqrt(sp.kk * Cc);
    double x0 = ceil(mx - hx - 0.5), x1 = floor(mx + hx - 0.5);
    double y0 = ceil(my - hy - 0.5), y1 = floor(my + hy - 0.5);
    x0 = fmax(x0, 0.0); y0 = fmax(y0, 0.0);
    x1 = fmin(x1, (double)(cam.W - 1)); y1 = fmin(y1, (double)(cam.H - 1));
    const bool keep = det > 0.0 && sp.o >= (1.0 / 255.0) && x0 <= x1 && y0 <= y1;

    // colour along the unit view direction
    double oc[3];
    for (int j = 0; j < 3; j++) oc[j] = -(Rc[0 * 3 + j] * tc[0] + Rc[1 * 3 + j] * tc[1] + Rc[2 * 3 + j] * tc[2]);
    const double v0 = sp.mu[0] - oc[0], v1 = sp.mu[1] - oc[1], v2 = sp.mu[2] - oc[2];
    const double vn = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
    double Y[16];
    sh_eval_basis(v0 / vn, v1 / vn, v2 / vn, DEG, Y);
    double col[3];
#pragma unroll
    for (int ch = 0; ch < 3; ch++) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < nk; k++) acc += Y[k] * (double)shv[k * 3 + ch];
        acc += 0.5;
        col[ch] = acc < 0.0 ? 0.0 : acc;
    }
    // The colour is masked with a lane mask the compiler cannot see
    // through (a select would be turned back into a branch around the
    // colour), so its loads and arithmetic stay in this block; a culled
    // entry keeps exact zeros.
    uint32_t km = keep ? 0xFFFFFFFFu : 0u;
    __asm__ __volatile__("" : "+v"(km));
    rr.rgb = make_float4(__uint_as_float(__float_as_uint((float)col[0]) & km),
                         __uint_as_float(__float_as_uint((float)col[1]) & km),
                         __uint_as_float(__float_as_uint((float)col[2]) & km), 0.f);
    if (!keep) return;

    const float mxh = (float)mx, myh = (float)my;
    rr.m = make_float4(mxh, myh, (float)(mx - (double)mxh), (float)(my - (double)myh));
    rr.c = make_float4((float)(Cc / det), (float)(-B / det), (float)(A / det), (float)sp.o);
    const int ix0 = (int)x0, iy0 = (int)y0, ix1 = (int)x1, iy1 = (int)y1;
    bx = make_short4((short)ix0, (short)iy0, (short)ix1, (short)iy1);
    // bins touched (the box lies in the image: no negative coordinates)
    nt = (uint32_t)(((ix1 >> bs) - (ix0 >> bs) + 1) * ((iy1 >> bs) - (iy0 >> bs) + 1));
}

template <int DEG, bool BUF>
__global__ void __launch_bounds__(256) k_project(const SceneTable sc, const ViewTable vt, BlendRec *__restrict__ rec,
                                                 uint32_t *__restrict__ depth_key, short4 *__restrict__ box,
                                                 uint32_t *__restrict__ ntiles, uint32_t *__restrict__ n_ent) {
    const int v = (int)(blockIdx.x % (unsigned)vt.n_views);
    const int64_t i = (int64_t)(blockIdx.x / (unsigned)vt.n_views) * blockDim.x + threadIdx.x;
    const GaussPtrs &g = sc.g[v];
    const DevCam &cam = vt.cam[v];
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_ent = (uint32_t)vt.ent_base[vt.n_views];
    if (i >= g.n) return;
    const int64_t n = g.n;
    const uint32_t bo = (uint32_t)i * 4u;   // the lane's byte offset in every parameter row
    const int64_t e = (int64_t)vt.ent_base[v] + i;
    double mu[3], s[3], q[4];
    for (int k = 0; k < 3; k++) mu[k] = (double)at_row(g.means, k, n, bo);
    for (int k = 0; k < 3; k++) s[k] = exp((double)at_row(g.log_scales, k, n, bo));
    for (int k = 0; k < 4; k++) q[k] = (double)at_row(g.quats, k, n, bo);
    const double ologit = (double)g.opac[i];

    double Rc[9], tc[3];
    for (int k = 0; k < 9; k++) Rc[k] = (double)cam.R[k];
    for (int k = 0; k < 3; k++) tc[k] = (double)cam.t[k];

    double tv[3];
    for (int r = 0; r < 3; r++) tv[r] = Rc[r * 3 + 0] * mu[0] + Rc[r * 3 + 1] * mu[1] + Rc[r * 3 + 2] * mu[2] + tc[r];
    const double tz = tv[2];
    depth_key[e] = __float_as_uint((float)tz);

    BlendRec rr;
    rr.m = make_float4(0.f, 0.f, 0.f, 0.f);
    rr.c = make_float4(0.f, 0.f, 0.f, 0.f);
    rr.rgb = make_float4(0.f, 0.f, 0.f, 0.f);
    short4 bx = make_short4(0, 0, -1, -1);
    uint32_t nt = 0;
    if (tz > AS_NEAR) {
        // The SH coefficients are loaded here, so their latency overlaps the
        // covariance and box arithmetic below (an entry culled after this
        // point has read them for nothing; in front of the camera few are).
        // One buffer resource over the array with the row's byte offset a
        // scalar, when every row offset fits 32 bits, else 64-bit row addresses.
        float shv[(DEG + 1) * (DEG + 1) * 3];
        load_sh<(DEG + 1) * (DEG + 1) * 3, BUF>(g, bo, shv);
        __asm__ __volatile__("" ::: "memory");   // the loads are issued here, not next to their use
        project_entry<DEG>(shape_of(mu, s, q, ologit), shv, cam, Rc, tc, tv, vt.bin_shift, rr, bx, nt);
    }
    rec[e] = rr;
    box[e] = bx;
    ntiles[e] = nt;
}

constexpr int64_t PRJ_BLOCKS = 1536;   // six blocks of four waves on each CU

// Views that share a Gaussian set, and the blocks of 256 of its Gaussians.
struct ViewGroups {
    int32_t n;
    uint32_t block0[AS_MAX_VIEWS + 1];
    int32_t first[AS_MAX_VIEWS];   // a view of the group
    int32_t next[AS_MAX_VIEWS];    // the group's next view (-1: none)
};

// Several views: one thread per Gaussian walks the views that show its set, so
// the exponentials, the logarithm and the covariance are taken once per
// Gaussian, not per entry: with a thread per entry this FP64 arithmetic bounded
// the launch (1116 instructions a wave).  Eight views of 1.5M Gaussians
// 508 -> 402 us, 16 of 500,000 340 -> 257 us, eight over four sets of 0.3M to 2M
// Gaussians 630 -> 314 us.  The SH coefficients are read again for each view, from cache.
template <int DEG, bool BUF>
__global__ void __launch_bounds__(256) k_project_views(const SceneTable sc, const ViewTable vt, const ViewGroups vg,
                                                       BlendRec *__restrict__ rec, uint32_t *__restrict__ depth_key,
                                                       short4 *__restrict__ box, uint32_t *__restrict__ ntiles,
                                                       uint32_t *__restrict__ n_ent) {
    int grp = 0;
    for (int k = 1; k < vg.n; k++) grp += blockIdx.x >= vg.block0[k] ? 1 : 0;
    const int64_t i = (int64_t)(blockIdx.x - vg.block0[grp]) * blockDim.x + threadIdx.x;
    const GaussPtrs &g = sc.g[vg.first[grp]];
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_ent = (uint32_t)vt.ent_base[vt.n_views];
    if (i >= g.n) return;
    const int64_t n = g.n;
    const uint32_t bo = (uint32_t)i * 4u;   // the lane's byte offset in every parameter row
    double mu[3], s[3], q[4];
    for (int k = 0; k < 3; k++) mu[k] = (double)at_row(g.means, k, n, bo);
    for (int k = 0; k < 3; k++) s[k] = exp((double)at_row(g.log_scales, k, n, bo));
    for (int k = 0; k < 4; k++) q[k] = (double)at_row(g.quats, k, n, bo);
    const Shape sp = shape_of(mu, s, q, (double)g.opac[i]);
    for (int v = vg.first[grp]; v >= 0; v = vg.next[v]) {
        // keeps the coefficients' loads inside the loop instead of 48 values
        // held in registers across it
        __asm__ __volatile__("" ::: "memory");
        const DevCam &cam = vt.cam[v];
        const int64_t e = (int64_t)vt.ent_base[v] + i;
        double Rc[9], tc[3], tv[3];
        for (int k = 0; k < 9; k++) Rc[k] = (double)cam.R[k];
        for (int k = 0; k < 3; k++) tc[k] = (double)cam.t[k];
        for (int r = 0; r < 3; r++)
            tv[r] = Rc[r * 3 + 0] * sp.mu[0] + Rc[r * 3 + 1] * sp.mu[1] + Rc[r * 3 + 2] * sp.mu[2] + tc[r];
        depth_key[e] = __float_as_uint((float)tv[2]);
        BlendRec rr;
        rr.m = make_float4(0.f, 0.f, 0.f, 0.f);
        rr.c = make_float4(0.f, 0.f, 0.f, 0.f);
        rr.rgb = make_float4(0.f, 0.f, 0.f, 0.f);
        short4 bx = make_short4(0, 0, -1, -1);
        uint32_t nt = 0;
        if (tv[2] > AS_NEAR) {
            float shv[(DEG + 1) * (DEG + 1) * 3];
            load_sh<(DEG + 1) * (DEG + 1) * 3, BUF>(g, bo, shv);
            __asm__ __volatile__("" ::: "memory");
            project_entry<DEG>(sp, shv, cam, Rc, tc, tv, vt.bin_shift, rr, bx, nt);
        }
        rec[e] = rr;
        box[e] = bx;
        ntiles[e] = nt;
    }
}

}  // namespace

void launch_project(const SceneTable &sc, const ViewTable &vt, int64_t max_n, int deg, BlendRec *rec,
                    uint32_t *depth_key, int16_t *box, uint32_t *ntiles, uint32_t *n_ent, hipStream_t s,
                    bool force_addr64) {
    if (max_n == 0 || vt.n_views == 0) {
        launch_fill_u32(n_ent, 0u, 1, s);
        return;
    }
    short4 *b4 = reinterpret_cast<short4 *>(box);
    // buffer addressing of the SH rows when the last row's byte offset fits 32 bits
    const bool buf = !force_addr64 && 3 * (int64_t)(deg + 1) * (deg + 1) * max_n * 4 <= (int64_t)UINT32_MAX;
    // One view takes the kernel that keeps fewer values live; views of one set
    // (as the caller names it: equal pointers) are walked together, but only as
    // many as leave the launch PRJ_BLOCKS blocks: 16 views of 36,000 Gaussians are 2256
    // blocks with a thread per entry and 141 with a thread per Gaussian.
    ViewGroups vg;
    memset(&vg, 0, sizeof(vg));
    int64_t entry_blocks = 0;
    for (int v = 0; v < vt.n_views; v++) entry_blocks += (sc.g[v].n + 255) / 256;
    const int64_t most = entry_blocks / PRJ_BLOCKS;
    int members[AS_MAX_VIEWS] = {0};
    for (int v = 0; v < vt.n_views; v++) {
        const GaussPtrs &a = sc.g[v];
        vg.next[v] = -1;
        int grp = 0;
        for (; grp < vg.n; grp++) {
            const GaussPtrs &b = sc.g[vg.first[grp]];
            if (a.means == b.means && a.log_scales == b.log_scales && a.quats == b.quats && a.opac == b.opac &&
                a.sh == b.sh && a.n == b.n && members[grp] < most)
                break;
        }
        members[grp]++;
        if (grp == vg.n) {
            vg.first[vg.n++] = v;
            vg.block0[vg.n] = vg.block0[vg.n - 1] + (uint32_t)((a.n + 255) / 256);
        } else {
            int w = vg.first[grp];
            while (vg.next[w] >= 0) w = vg.next[w];
            vg.next[w] = v;
        }
    }
    // (sets of uneven sizes too: there the entry kernel's grid, max_n Gaussians
    // for every view, is mostly empty blocks)
    const bool views = vg.n < vt.n_views || 4 * entry_blocks < 3 * ((max_n + 255) / 256) * vt.n_views;
    const int64_t blocks = views ? (int64_t)vg.block0[vg.n] : (max_n + 255) / 256 * vt.n_views;
#define AS_PRJ(D, B)                                                                                               \
    do {                                                                                                           \
        if (views) hipLaunchKernelGGL((k_project_views<D, B>), dim3((unsigned)blocks), dim3(256), 0, s, sc, vt,    \
                                      vg, rec, depth_key, b4, ntiles, n_ent);                                      \
        else hipLaunchKernelGGL((k_project<D, B>), dim3((unsigned)blocks), dim3(256), 0, s, sc, vt, rec,           \
                                depth_key, b4, ntiles, n_ent);                                                     \
    } while (0)
    switch (deg) {
    case 0: if (buf) AS_PRJ(0, true); else AS_PRJ(0, false); break;
    case 1: if (buf) AS_PRJ(1, true); else AS_PRJ(1, false); break;
    case 2: if (buf) AS_PRJ(2, true); else AS_PRJ(2, false); break;
    default: if (buf) AS_PRJ(3, true); else AS_PRJ(3, false); break;
    }
#undef AS_PRJ
}

AS_WARM_KERNEL(project)
