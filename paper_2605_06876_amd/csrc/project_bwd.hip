// Reverse pass of the projection (Sec. 3): from the per-entry 2D gradients
// (mean, conic, opacity, colour) accumulated by the blend back to the stored
// parameters (means, log-scales, quaternions, opacity logits, SH).  One thread
// per Gaussian, FP64, struct-of-arrays reads and writes.  A batch of views is
// one launch: each thread walks the views in order and sums their
// contributions (a fixed order, so the sum is deterministic), then writes
// every gradient once.  A single view uses a leaner kernel.  Both follow the
// same chain in FP64, but the several-view kernel regroups it (contracted
// multiply-adds, shared reciprocals, one direction gradient of the channels'
// summed coefficients), so their results differ by FP64 rounding.
//
// Chain: colour = max(0, sum_k Y_k(d) sh_k + 1/2) with d = (mu - o_v)/|mu - o_v|;
// mean2d = (fx tx/tz + cx, fy ty/tz + cy); conic = inverse(J W Sigma W^T J^T
// + 0.3 I) with J the perspective Jacobian at the clamped centre; Sigma =
// R(q/|q|) diag(exp(2 log s)) R^T; o = sigmoid(logit).  The scale and
// rotation gradients are linear in dL/dSigma, so dL/dSigma is summed over the
// views first and mapped to (log s, q) once.
#include "internal.h"
#include "sh_device.h"

namespace {

// SH rows of the single-view kernel.  With BUF (every row offset of the
// array below 2^32 bytes: 48 rows of fewer than 22M Gaussians) a row is read
// and written through one buffer resource over the array, the row's byte
// offset a scalar and the lane's offset the one vector operand shared by all
// rows; otherwise through at_row.  A 64-bit address per row would be held in
// vector registers otherwise: the 48 rows' reads and writes took the kernel
// to 239 VGPRs, two waves per SIMD.
template <bool BUF>
__device__ __forceinline__ float sh_ld(const float *a, int row, int64_t n, uint32_t bo) {
    if constexpr (BUF) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a), (short)0, -1,
                                                                            AS_BUFFER_RSRC_WORD3);
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)bo, (int)((uint32_t)row * (uint32_t)n * 4u), 0));
    } else {
        return at_row(a, row, n, bo);
    }
}
template <bool BUF>
__device__ __forceinline__ void sh_st(float *a, int row, int64_t n, uint32_t bo, float v) {
    if constexpr (BUF) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(a, (short)0, -1, AS_BUFFER_RSRC_WORD3);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)bo, (int)((uint32_t)row * (uint32_t)n * 4u), 0);
    } else {
        at_row(a, row, n, bo) = v;
    }
}

// One view: the form that keeps the fewest values live, used when a render
// has one view.
template <int DEG, bool BUF>
__global__ void __launch_bounds__(256) k_project_bwd_view(GaussPtrs g, DevCam cam, const uint32_t *__restrict__ ntiles,
                                                     const float *__restrict__ g2d, GradPtrs out,
                                                     float *__restrict__ g2d_norm, int32_t *__restrict__ vis_count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    const int64_t n = g.n, os = out.stride;
    const uint32_t bo = (uint32_t)i * 4u;   // the lane's byte offset in every row (n < 2^30)
    constexpr int nk = (DEG + 1) * (DEG + 1);
    if (ntiles[i] == 0) {
        for (int k = 0; k < 3; k++) { at_row(out.means, k, os, bo) = 0.f; at_row(out.log_scales, k, os, bo) = 0.f; }
        for (int k = 0; k < 4; k++) at_row(out.quats, k, os, bo) = 0.f;
        out.opac[i] = 0.f;
#pragma unroll
        for (int k = 0; k < nk * 3; k++) sh_st<BUF>(out.sh, k, os, bo, 0.f);
        return;
    }
    // The colour part first, from the mean and the colour gradient alone, and
    // a compiler barrier before the rest is loaded: the geometry's inputs and
    // intermediates are not held in registers across the SH loops (together
    // they needed 236 VGPRs, two waves per SIMD).
    double mu[3];
    for (int k = 0; k < 3; k++) mu[k] = (double)at_row(g.means, k, n, bo);
    double Rc[9], tc[3];
    for (int k = 0; k < 9; k++) Rc[k] = (double)cam.R[k];
    for (int k = 0; k < 3; k++) tc[k] = (double)cam.t[k];
    double dmu[3];
    {
        const double grgb[3] = {g2d[i * 9 + 6], g2d[i * 9 + 7], g2d[i * 9 + 8]};
        // colour and view direction
        double oc[3];
        for (int j = 0; j < 3; j++) oc[j] = -(Rc[0 * 3 + j] * tc[0] + Rc[1 * 3 + j] * tc[1] + Rc[2 * 3 + j] * tc[2]);
        const double v[3] = {mu[0] - oc[0], mu[1] - oc[1], mu[2] - oc[2]};
        const double vn = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        const double d[3] = {v[0] / vn, v[1] / vn, v[2] / vn};
        double Y[16];
        sh_eval_basis(d[0], d[1], d[2], DEG, Y);
        // One pass over the coefficients: per channel the raw colour
        // sum_k Y_k sh_k (its clamp decides whether the channel's gradient
        // passes) and the gradient of that sum with respect to the direction,
        // G_ch = sum_k sh_k dY_k (the terms of sh_weighted_grad).  The
        // direction gradient is then sum_ch gc_ch G_ch, the same sum as
        // sum_k (sum_ch sh_k gc_ch) dY_k regrouped, so the coefficients are not
        // read a second time (a second read missed L2 and cost about 100 MB of
        // HBM traffic per C2 launch).
        double gc[3], gd[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            double shc[16], raw = 0.0;
#pragma unroll
            for (int k = 0; k < nk; k++) {
                shc[k] = (double)sh_ld<BUF>(g.sh, k * 3 + ch, n, bo);
                raw += Y[k] * shc[k];
            }
            double gch[3];
            sh_weighted_grad(d[0], d[1], d[2], DEG, shc, gch);
            gc[ch] = raw + 0.5 < 0.0 ? 0.0 : grgb[ch];
            for (int a = 0; a < 3; a++) gd[a] += gc[ch] * gch[a];
        }
#pragma unroll
        for (int k = 0; k < nk; k++)
#pragma unroll
            for (int ch = 0; ch < 3; ch++) sh_st<BUF>(out.sh, k * 3 + ch, os, bo, (float)(Y[k] * gc[ch]));
        const double ddot = gd[0] * d[0] + gd[1] * d[1] + gd[2] * d[2];
        for (int a = 0; a < 3; a++) dmu[a] = (gd[a] - d[a] * ddot) / vn;
    }
    // the colour part's result is an operand of the barrier, so its arithmetic
    // finishes before the geometry's loads, which the barrier holds after it
    __asm__ __volatile__("" : "+v"(dmu[0]), "+v"(dmu[1]), "+v"(dmu[2]) : : "memory");

    const double gm0 = g2d[i * 9 + 0], gm1 = g2d[i * 9 + 1];
    const double gca = g2d[i * 9 + 2], gcb = g2d[i * 9 + 3], gcc = g2d[i * 9 + 4];
    const double gop = g2d[i * 9 + 5];
    if (g2d_norm) g2d_norm[i] += (float)sqrt(gm0 * gm0 + gm1 * gm1);
    if (vis_count) vis_count[i] += 1;
    double s[3], q[4];
    for (int k = 0; k < 3; k++) s[k] = exp((double)at_row(g.log_scales, k, n, bo));
    for (int k = 0; k < 4; k++) q[k] = (double)at_row(g.quats, k, n, bo);
    const double o = 1.0 / (1.0 + exp(-(double)g.opac[i]));
    const double fx = cam.fx, fy = cam.fy;
    double tv[3];
    for (int r = 0; r < 3; r++) tv[r] = Rc[r * 3 + 0] * mu[0] + Rc[r * 3 + 1] * mu[1] + Rc[r * 3 + 2] * mu[2] + tc[r];
    const double tx = tv[0], ty = tv[1], tz = tv[2];
    const double qnorm = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double w = q[0] / qnorm, x = q[1] / qnorm, y = q[2] / qnorm, z = q[3] / qnorm;
    const double Rg[9] = {1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y),
                          2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x),
                          2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)};
    // opacity
    out.opac[i] = (float)(gop * o * (1.0 - o));

    // mean2d
    double dt[3] = {0.0, 0.0, 0.0};
    dt[0] += gm0 * fx / tz;
    dt[1] += gm1 * fy / tz;
    dt[2] += -gm0 * fx * tx / (tz * tz) - gm1 * fy * ty / (tz * tz);

    // conic = inverse(cov): dL/dcov = -K G K
    const double limx = 1.3 * ((double)cam.W / (2.0 * fx));
    const double limy = 1.3 * ((double)cam.H / (2.0 * fy));
    const double txtz = tx / tz, tytz = ty / tz;
    const bool clx = txtz < -limx || txtz > limx, cly = tytz < -limy || tytz > limy;
    const double cx_ = fmin(limx, fmax(-limx, txtz)) * tz;
    const double cy_ = fmin(limy, fmax(-limy, tytz)) * tz;
    const double J[6] = {fx / tz, 0.0, -(fx * cx_) / (tz * tz), 0.0, fy / tz, -(fy * cy_) / (tz * tz)};
    double T[6];
    for (int r = 0; r < 2; r++)
        for (int k = 0; k < 3; k++)
            T[r * 3 + k] = J[r * 3 + 0] * Rc[k] + J[r * 3 + 1] * Rc[3 + k] + J[r * 3 + 2] * Rc[6 + k];
    double Sg[9];
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            double acc = 0.0;
            for (int k = 0; k < 3; k++) acc += Rg[a * 3 + k] * (s[k] * s[k]) * Rg[b * 3 + k];
            Sg[a * 3 + b] = acc;
        }
    double C2[4];
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) {
            double acc = 0.0;
            for (int k = 0; k < 3; k++)
                for (int l = 0; l < 3; l++) acc += T[a * 3 + k] * Sg[k * 3 + l] * T[b * 3 + l];
            C2[a * 2 + b] = acc;
        }
    const double A = C2[0] + AS_LOWPASS, B = C2[1], Cc = C2[3] + AS_LOWPASS;
    const double det = A * Cc - B * B;
    const double K[4] = {Cc / det, -B / det, -B / det, A / det};
    const double Gk[4] = {gca, 0.5 * gcb, 0.5 * gcb, gcc};
    double KG[4], Gc[4];
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) KG[a * 2 + b] = K[a * 2] * Gk[b] + K[a * 2 + 1] * Gk[2 + b];
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) Gc[a * 2 + b] = -(KG[a * 2] * K[b] + KG[a * 2 + 1] * K[2 + b]);
    double dS[9], dT[6];
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            double acc = 0.0;
            for (int r = 0; r < 2; r++)
                for (int qq = 0; qq < 2; qq++) acc += T[r * 3 + a] * Gc[r * 2 + qq] * T[qq * 3 + b];
            dS[a * 3 + b] = acc;
        }
    for (int r = 0; r < 2; r++)
        for (int k = 0; k < 3; k++) {
            double acc = 0.0;
            for (int qq = 0; qq < 2; qq++)
                for (int l = 0; l < 3; l++) acc += Gc[r * 2 + qq] * T[qq * 3 + l] * Sg[l * 3 + k];
            dT[r * 3 + k] = 2.0 * acc;
        }
    double dJ[6];
    for (int r = 0; r < 2; r++)
        for (int k = 0; k < 3; k++)
            dJ[r * 3 + k] = dT[r * 3 + 0] * Rc[k * 3 + 0] + dT[r * 3 + 1] * Rc[k * 3 + 1] + dT[r * 3 + 2] * Rc[k * 3 + 2];
    dt[2] += dJ[0] * (-fx / (tz * tz)) + dJ[4] * (-fy / (tz * tz));
    if (!clx) {
        dt[0] += dJ[2] * (-fx / (tz * tz));
        dt[2] += dJ[2] * (2.0 * fx * tx / (tz * tz * tz));
    } else {
        dt[2] += dJ[2] * (fx * (cx_ / tz) / (tz * tz));
    }
    if (!cly) {
        dt[1] += dJ[5] * (-fy / (tz * tz));
        dt[2] += dJ[5] * (2.0 * fy * ty / (tz * tz * tz));
    } else {
        dt[2] += dJ[5] * (fy * (cy_ / tz) / (tz * tz));
    }
    for (int a = 0; a < 3; a++) dmu[a] += Rc[0 * 3 + a] * dt[0] + Rc[1 * 3 + a] * dt[1] + Rc[2 * 3 + a] * dt[2];
    for (int a = 0; a < 3; a++) at_row(out.means, a, os, bo) = (float)dmu[a];
    // scales
    for (int k = 0; k < 3; k++) {
        double acc = 0.0;
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++) acc += Rg[a * 3 + k] * dS[a * 3 + b] * Rg[b * 3 + k];
        at_row(out.log_scales, k, os, bo) = (float)(2.0 * s[k] * s[k] * acc);
    }
    // rotation -> quaternion
    double dR[9];
    for (int a = 0; a < 3; a++)
        for (int k = 0; k < 3; k++) {
            double acc = 0.0;
            for (int b = 0; b < 3; b++) acc += dS[a * 3 + b] * Rg[b * 3 + k];
            dR[a * 3 + k] = 2.0 * acc * s[k] * s[k];
        }
    double dq[4];
    dq[0] = 2.0 * (-z * dR[1] + y * dR[2] + z * dR[3] - x * dR[5] - y * dR[6] + x * dR[7]);
    dq[1] = 2.0 * (y * dR[1] + z * dR[2] + y * dR[3] - 2.0 * x * dR[4] - w * dR[5] + z * dR[6] + w * dR[7] -
                   2.0 * x * dR[8]);
    dq[2] = 2.0 * (-2.0 * y * dR[0] + x * dR[1] + w * dR[2] + x * dR[3] + z * dR[5] - w * dR[6] + z * dR[7] -
                   2.0 * y * dR[8]);
    dq[3] = 2.0 * (-2.0 * z * dR[0] - w * dR[1] + x * dR[2] + w * dR[3] - 2.0 * z * dR[4] + y * dR[5] + x * dR[6] +
                   y * dR[7]);
    const double qn[4] = {w, x, y, z};
    const double qd = dq[0] * w + dq[1] * x + dq[2] * y + dq[3] * z;
    for (int k = 0; k < 4; k++) at_row(out.quats, k, os, bo) = (float)((dq[k] - qn[k] * qd) / qnorm);
}


// A row of the world-to-view transform, rounded as in the forward pass (which
// decides the clamp of the Jacobian's centre on it).
__device__ __forceinline__ double view_row(const double *R, const double mu[3], double t) {
#pragma clang fp contract(off)
    return R[0] * mu[0] + R[1] * mu[1] + R[2] * mu[2] + t;
}

// All views of a batch in one pass per Gaussian (SH rows addressed as in the
// single-view kernel, BUF).
//
// Bound by its FP64 instructions and, at few waves, their latency.  So a view
// costs as few of them as the chain needs: Sigma is taken once, products with
// the 2x3 T are formed once and reused (T Sigma gives the covariance and
// dL/dT), symmetric results have their six or three terms, divisions by tz,
// |v| and det are one reciprocal each, and the three channels share one
// direction gradient of the summed coefficients.  What is not needed from
// view to view (rotation, scales) is loaded and formed again after the loop; the SH
// coefficients stay in registers as floats, their gradients in LDS, the next
// view's 2D gradients are on their way: two waves per SIMD instead of one.
// Eight views of 1.5M Gaussians 1020 -> 460 us (its 1.2 GB 250 us at a copy's
// rate, its instructions 280).  Three waves spill: 2030 us; LDS float atomics
// for the SH gradients, every lane its own word: 2860 us (2.5 cycles a lane).
template <int DEG, bool BUF>
__global__ void __launch_bounds__(256, 2) k_project_bwd(GaussPtrs g, const ViewTable vt,
                                                        const uint32_t *__restrict__ ntiles,
                                                        const float *__restrict__ g2d, GradPtrs out,
                                                        float *__restrict__ g2d_norm, int32_t *__restrict__ vis_count) {
#pragma clang fp contract(fast)
    constexpr int nk = (DEG + 1) * (DEG + 1);
    // SH gradient accumulators live in LDS (thread-private columns), not registers
    __shared__ float s_dsh[nk * 3][256];
    const int tid = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + tid;
    if (i >= g.n) return;
    const int64_t n = g.n, os = out.stride;
    const uint32_t bo = (uint32_t)i * 4u;   // the lane's byte offset in every row
#pragma unroll
    for (int k = 0; k < nk * 3; k++) s_dsh[k][tid] = 0.f;

    struct Rot {
        double R[9], q[4], norm;
    };
    auto rotation = [&]() {
        Rot r;
        double q[4];
        for (int k = 0; k < 4; k++) q[k] = (double)at_row(g.quats, k, n, bo);
        r.norm = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
        for (int k = 0; k < 4; k++) r.q[k] = q[k] / r.norm;
        const double w = r.q[0], x = r.q[1], y = r.q[2], z = r.q[3];
        r.R[0] = 1.0 - 2.0 * (y * y + z * z), r.R[1] = 2.0 * (x * y - w * z), r.R[2] = 2.0 * (x * z + w * y);
        r.R[3] = 2.0 * (x * y + w * z), r.R[4] = 1.0 - 2.0 * (x * x + z * z), r.R[5] = 2.0 * (y * z - w * x);
        r.R[6] = 2.0 * (x * z - w * y), r.R[7] = 2.0 * (y * z + w * x), r.R[8] = 1.0 - 2.0 * (x * x + y * y);
        return r;
    };
    double mu[3];
    for (int k = 0; k < 3; k++) mu[k] = (double)at_row(g.means, k, n, bo);
    // Sigma, symmetric: xx, xy, xz, yy, yz, zz
    double S0, S1, S2, S3, S4, S5;
    {
        const Rot r = rotation();
        double s2[3];
        for (int k = 0; k < 3; k++) {
            const double sk = exp((double)at_row(g.log_scales, k, n, bo));
            s2[k] = sk * sk;
        }
        auto sig = [&](int a, int b) {
            return r.R[3 * a] * s2[0] * r.R[3 * b] + r.R[3 * a + 1] * s2[1] * r.R[3 * b + 1] +
                   r.R[3 * a + 2] * s2[2] * r.R[3 * b + 2];
        };
        S0 = sig(0, 0), S1 = sig(0, 1), S2 = sig(0, 2), S3 = sig(1, 1), S4 = sig(1, 2), S5 = sig(2, 2);
    }
    float shv[nk * 3];
#pragma unroll
    for (int k = 0; k < nk * 3; k++) shv[k] = sh_ld<BUF>(g.sh, k, n, bo);

    double dmu[3] = {0.0, 0.0, 0.0};
    double D0 = 0.0, D1 = 0.0, D2 = 0.0, D3 = 0.0, D4 = 0.0, D5 = 0.0;   // dL/dSigma, laid out as Sigma
    double gop = 0.0;
    float nrm = 0.f;
    int32_t vis = 0;

    // the 2D gradients of a view, one view ahead
    float gq[9];
    uint32_t nt_next = 0;
    auto fetch = [&](int v) {
        const int64_t e = (int64_t)vt.ent_base[v] + i;
        nt_next = ntiles[e];
#pragma unroll
        for (int k = 0; k < 9; k++) gq[k] = g2d[e * 9 + k];
    };
    fetch(0);
    for (int v = 0; v < vt.n_views; v++) {
        const uint32_t nt = nt_next;
        const double gm0 = gq[0], gm1 = gq[1], gca = gq[2], gcb = gq[3], gcc = gq[4], go = gq[5];
        const double grgb[3] = {gq[6], gq[7], gq[8]};
        if (v + 1 < vt.n_views) fetch(v + 1);
        if (nt == 0) continue;
        // the coefficients are widened where they are used, not once for the
        // whole loop (96 registers)
#pragma unroll
        for (int k = 0; k < nk * 3; k++) __asm__ __volatile__("" : "+v"(shv[k]));
        const DevCam &cam = vt.cam[v];
        gop += go;
        nrm += (float)sqrt(gm0 * gm0 + gm1 * gm1);
        vis += 1;

        double Rc[9], tc[3];
        for (int k = 0; k < 9; k++) Rc[k] = (double)cam.R[k];
        for (int k = 0; k < 3; k++) tc[k] = (double)cam.t[k];
        double tv[3];
        for (int r = 0; r < 3; r++) tv[r] = view_row(&Rc[3 * r], mu, tc[r]);
        const double tx = tv[0], ty = tv[1], tz = tv[2], itz = 1.0 / tz;
        const double fxz = cam.fx * itz, fyz = cam.fy * itz;

        // the clamp of the Jacobian's centre is decided as in the forward pass
        const double limx = 1.3 * ((double)cam.W / (2.0 * (double)cam.fx));
        const double limy = 1.3 * ((double)cam.H / (2.0 * (double)cam.fy));
        const double txtz = tx / tz, tytz = ty / tz;
        const bool clx = txtz < -limx || txtz > limx, cly = tytz < -limy || tytz > limy;
        const double ux = fmin(limx, fmax(-limx, txtz)), uy = fmin(limy, fmax(-limy, tytz));
        // T = J Rc with J = (fx/tz, 0, -fx ux/tz; 0, fy/tz, -fy uy/tz)
        const double j2 = -fxz * ux, j5 = -fyz * uy;
        double T0[3], T1[3];
        for (int k = 0; k < 3; k++) {
            T0[k] = fxz * Rc[k] + j2 * Rc[6 + k];
            T1[k] = fyz * Rc[3 + k] + j5 * Rc[6 + k];
        }
        const double M0[3] = {T0[0] * S0 + T0[1] * S1 + T0[2] * S2, T0[0] * S1 + T0[1] * S3 + T0[2] * S4,
                              T0[0] * S2 + T0[1] * S4 + T0[2] * S5};
        const double M1[3] = {T1[0] * S0 + T1[1] * S1 + T1[2] * S2, T1[0] * S1 + T1[1] * S3 + T1[2] * S4,
                              T1[0] * S2 + T1[1] * S4 + T1[2] * S5};
        const double A = M0[0] * T0[0] + M0[1] * T0[1] + M0[2] * T0[2] + AS_LOWPASS;
        const double B = M0[0] * T1[0] + M0[1] * T1[1] + M0[2] * T1[2];
        const double C = M1[0] * T1[0] + M1[1] * T1[1] + M1[2] * T1[2] + AS_LOWPASS;
        // conic = inverse(cov): dL/dcov = -K G K
        const double idet = 1.0 / (A * C - B * B);
        const double K0 = C * idet, K1 = -B * idet, K2 = A * idet, gh = 0.5 * gcb;
        const double a00 = K0 * gca + K1 * gh, a01 = K0 * gh + K1 * gcc, a10 = K1 * gca + K2 * gh,
                     a11 = K1 * gh + K2 * gcc;
        const double G0 = -(a00 * K0 + a01 * K1), G1 = -(a00 * K1 + a01 * K2), G2 = -(a10 * K1 + a11 * K2);
        double P0[3], P1[3], dT0[3], dT1[3];
        for (int k = 0; k < 3; k++) {
            P0[k] = G0 * T0[k] + G1 * T1[k];
            P1[k] = G1 * T0[k] + G2 * T1[k];
            dT0[k] = 2.0 * (G0 * M0[k] + G1 * M1[k]);
            dT1[k] = 2.0 * (G1 * M0[k] + G2 * M1[k]);
        }
        D0 += T0[0] * P0[0] + T1[0] * P1[0];
        D1 += T0[0] * P0[1] + T1[0] * P1[1];
        D2 += T0[0] * P0[2] + T1[0] * P1[2];
        D3 += T0[1] * P0[1] + T1[1] * P1[1];
        D4 += T0[1] * P0[2] + T1[1] * P1[2];
        D5 += T0[2] * P0[2] + T1[2] * P1[2];
        const double dJ0 = dT0[0] * Rc[0] + dT0[1] * Rc[1] + dT0[2] * Rc[2];
        const double dJ2 = dT0[0] * Rc[6] + dT0[1] * Rc[7] + dT0[2] * Rc[8];
        const double dJ4 = dT1[0] * Rc[3] + dT1[1] * Rc[4] + dT1[2] * Rc[5];
        const double dJ5 = dT1[0] * Rc[6] + dT1[1] * Rc[7] + dT1[2] * Rc[8];
        // mean2d = (fx tx/tz, fy ty/tz), then J
        double dt0 = gm0 * fxz, dt1 = gm1 * fyz;
        double dt2 = -(dt0 * tx + dt1 * ty + dJ0 * fxz + dJ4 * fyz) * itz;
        const double ex = dJ2 * fxz * itz, ey = dJ5 * fyz * itz;
        if (!clx) {
            dt0 -= ex;
            dt2 += 2.0 * ex * txtz;
        } else {
            dt2 += ex * ux;
        }
        if (!cly) {
            dt1 -= ey;
            dt2 += 2.0 * ey * tytz;
        } else {
            dt2 += ey * uy;
        }
        for (int k = 0; k < 3; k++) dmu[k] += Rc[k] * dt0 + Rc[3 + k] * dt1 + Rc[6 + k] * dt2;

        // colour and view direction: the raw colour decides each channel's
        // clamp, the channels' gradients weight the coefficients, and those
        // give the direction gradient
        double d[3], Y[16];
        for (int j = 0; j < 3; j++) d[j] = mu[j] + (Rc[0 * 3 + j] * tc[0] + Rc[1 * 3 + j] * tc[1] + Rc[2 * 3 + j] * tc[2]);
        const double ivn = 1.0 / sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        for (int j = 0; j < 3; j++) d[j] *= ivn;
        sh_eval_basis(d[0], d[1], d[2], DEG, Y);
        double gc[3], wk[16], gd[3];
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            double raw = 0.0;
#pragma unroll
            for (int k = 0; k < nk; k++) raw += Y[k] * (double)shv[k * 3 + ch];
            gc[ch] = raw + 0.5 < 0.0 ? 0.0 : grgb[ch];
        }
#pragma unroll
        for (int k = 0; k < nk; k++) {
            wk[k] = gc[0] * (double)shv[k * 3] + gc[1] * (double)shv[k * 3 + 1] + gc[2] * (double)shv[k * 3 + 2];
#pragma unroll
            for (int ch = 0; ch < 3; ch++) s_dsh[k * 3 + ch][tid] += (float)(Y[k] * gc[ch]);
        }
        sh_weighted_grad(d[0], d[1], d[2], DEG, wk, gd);
        const double ddot = gd[0] * d[0] + gd[1] * d[1] + gd[2] * d[2];
        for (int k = 0; k < 3; k++) dmu[k] += (gd[k] - d[k] * ddot) * ivn;
    }

    if (vis && g2d_norm) g2d_norm[i] += nrm;
    if (vis && vis_count) vis_count[i] += vis;
    if (!vis) {   // no view saw it: zero gradients
        for (int k = 0; k < 3; k++) { at_row(out.means, k, os, bo) = 0.f; at_row(out.log_scales, k, os, bo) = 0.f; }
        for (int k = 0; k < 4; k++) at_row(out.quats, k, os, bo) = 0.f;
        out.opac[i] = 0.f;
#pragma unroll
        for (int k = 0; k < nk * 3; k++) sh_st<BUF>(out.sh, k, os, bo, 0.f);
        return;
    }
    __asm__ __volatile__("" ::: "memory");   // the parameters are loaded again, not held across the loop
    const double o = 1.0 / (1.0 + exp(-(double)g.opac[i]));
    out.opac[i] = (float)(gop * o * (1.0 - o));
#pragma unroll
    for (int k = 0; k < nk * 3; k++) sh_st<BUF>(out.sh, k, os, bo, s_dsh[k][tid]);
    for (int a = 0; a < 3; a++) at_row(out.means, a, os, bo) = (float)dmu[a];
    const Rot rot = rotation();
    const double *Rg = rot.R;
    double s2[3];
    for (int k = 0; k < 3; k++) {
        const double sk = exp((double)at_row(g.log_scales, k, n, bo));
        s2[k] = sk * sk;
    }
    // dR = 2 dSigma R diag(s^2); the scales' gradient is its projection on R
    double dR[9];
    for (int k = 0; k < 3; k++) {
        const double r0 = Rg[k], r1 = Rg[3 + k], r2 = Rg[6 + k];
        const double e0 = D0 * r0 + D1 * r1 + D2 * r2, e1 = D1 * r0 + D3 * r1 + D4 * r2, e2 = D2 * r0 + D4 * r1 + D5 * r2;
        at_row(out.log_scales, k, os, bo) = (float)(2.0 * s2[k] * (r0 * e0 + r1 * e1 + r2 * e2));
        dR[k] = 2.0 * e0 * s2[k];
        dR[3 + k] = 2.0 * e1 * s2[k];
        dR[6 + k] = 2.0 * e2 * s2[k];
    }
    // rotation -> quaternion
    const double w = rot.q[0], x = rot.q[1], y = rot.q[2], z = rot.q[3];
    double dq[4];
    dq[0] = 2.0 * (-z * dR[1] + y * dR[2] + z * dR[3] - x * dR[5] - y * dR[6] + x * dR[7]);
    dq[1] = 2.0 * (y * dR[1] + z * dR[2] + y * dR[3] - 2.0 * x * dR[4] - w * dR[5] + z * dR[6] + w * dR[7] -
                   2.0 * x * dR[8]);
    dq[2] = 2.0 * (-2.0 * y * dR[0] + x * dR[1] + w * dR[2] + x * dR[3] + z * dR[5] - w * dR[6] + z * dR[7] -
                   2.0 * y * dR[8]);
    dq[3] = 2.0 * (-2.0 * z * dR[0] - w * dR[1] + x * dR[2] + w * dR[3] - 2.0 * z * dR[4] + y * dR[5] + x * dR[6] +
                   y * dR[7]);
    const double qd = dq[0] * w + dq[1] * x + dq[2] * y + dq[3] * z;
    for (int k = 0; k < 4; k++) at_row(out.quats, k, os, bo) = (float)((dq[k] - rot.q[k] * qd) / rot.norm);
}

}  // namespace

void launch_project_bwd(const GaussPtrs &g, const ViewTable &vt, const uint32_t *ntiles, const float *grad2d,
                        GradPtrs out, float *g2d_norm, int32_t *vis_count, hipStream_t s, bool force_addr64) {
    if (g.n == 0) return;
    const dim3 grid((unsigned)((g.n + 255) / 256));
    // buffer addressing when the last SH row's byte offset fits 32 bits
    const int64_t rows = 3 * (int64_t)(g.deg + 1) * (g.deg + 1);
    const bool buf = !force_addr64 && rows * (g.n > out.stride ? g.n : out.stride) * 4 <= (int64_t)UINT32_MAX;
    if (vt.n_views == 1) {
        const DevCam &cam = vt.cam[0];
#define AS_PBV(D)                                                                                                  \
    do {                                                                                                           \
        if (buf) hipLaunchKernelGGL((k_project_bwd_view<D, true>), grid, dim3(256), 0, s, g, cam, ntiles, grad2d,  \
                                    out, g2d_norm, vis_count);                                                     \
        else hipLaunchKernelGGL((k_project_bwd_view<D, false>), grid, dim3(256), 0, s, g, cam, ntiles, grad2d, out, \
                                g2d_norm, vis_count);                                                              \
    } while (0)
        switch (g.deg) {
        case 0: AS_PBV(0); break;
        case 1: AS_PBV(1); break;
        case 2: AS_PBV(2); break;
        default: AS_PBV(3); break;
        }
#undef AS_PBV
        return;
    }
#define AS_PBB(D)                                                                                                  \
    do {                                                                                                           \
        if (buf) hipLaunchKernelGGL((k_project_bwd<D, true>), grid, dim3(256), 0, s, g, vt, ntiles, grad2d, out,   \
                                    g2d_norm, vis_count);                                                          \
        else hipLaunchKernelGGL((k_project_bwd<D, false>), grid, dim3(256), 0, s, g, vt, ntiles, grad2d, out,      \
                                g2d_norm, vis_count);                                                              \
    } while (0)
    switch (g.deg) {
    case 0: AS_PBB(0); break;
    case 1: AS_PBB(1); break;
    case 2: AS_PBB(2); break;
    default: AS_PBB(3); break;
    }
#undef AS_PBB
}

AS_WARM_KERNEL(project_bwd)
