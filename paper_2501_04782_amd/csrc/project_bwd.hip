// Adjoint of the EWA projection.  Per (frame, Gaussian) it sums the
// per-(Gaussian, tile) partials left by the compositing adjoint (contiguous
// slots of this Gaussian, in FP64), takes the conic of the forward record,
// re-derives the rest of the frame's projection and applies the chain rule down
// to the stored parameters in FP32; the shared parameters are summed over the
// frames in FP64.
// Each frame's pose gradient (dL/dRc, dL/dtc) is reduced per workgroup in a
// fixed order; a second kernel sums the workgroups and maps it to the 7-vector
// pose.  Everything is deterministic (no floating-point atomics).
#include "gv_internal.h"

namespace gv {

// dR_e * dR_e/dq for the e-th entry (row-major) of the rotation matrix of the
// unit quaternion (w, x, y, z); e is a compile-time constant after unrolling.
template <typename F>
__device__ __forceinline__ void add_rot_partial(int e, F v, const F q[4], F g[4]) {
    const F w = q[0], x = q[1], y = q[2], z = q[3];
    switch (e) {
        case 0: g[2] += -F(4) * y * v; g[3] += -F(4) * z * v; break;
        case 1: g[0] += -F(2) * z * v; g[1] += F(2) * y * v; g[2] += F(2) * x * v; g[3] += -F(2) * w * v; break;
        case 2: g[0] += F(2) * y * v; g[1] += F(2) * z * v; g[2] += F(2) * w * v; g[3] += F(2) * x * v; break;
        case 3: g[0] += F(2) * z * v; g[1] += F(2) * y * v; g[2] += F(2) * x * v; g[3] += F(2) * w * v; break;
        case 4: g[1] += -F(4) * x * v; g[3] += -F(4) * z * v; break;
        case 5: g[0] += -F(2) * x * v; g[1] += -F(2) * w * v; g[2] += F(2) * z * v; g[3] += F(2) * y * v; break;
        case 6: g[0] += -F(2) * y * v; g[1] += F(2) * z * v; g[2] += -F(2) * w * v; g[3] += F(2) * x * v; break;
        case 7: g[0] += F(2) * x * v; g[1] += F(2) * w * v; g[2] += F(2) * z * v; g[3] += F(2) * y * v; break;
        default: g[1] += -F(4) * x * v; g[2] += -F(4) * y * v; break;
    }
}

// FP32 quantities of the projection of (f, g) that the adjoint needs.  The
// conic is read from the forward record (the FP64 value rounded once: exactly
// the one the compositing kernels used); the rest is recomputed.
struct AdjIn {
    float mu[3], s[3], qh[4], iqn, R[9], Sig[6], m[3], iz, T[6], A[3], o;
    float N[4];  // B-spline weights of control points span .. span + 3
    int span;
};

// Cubic polynomial in t without a constant term: c1 t + c2 t^2 + c3 t^3.
template <typename T>
__device__ __forceinline__ float cubic_in_t(const Args& a, const void* coeffs, int rows, int k, int64_t g, float t) {
    const int64_t n = a.n;
    const float c1 = static_cast<float>(load_param<T>(coeffs, (0 * rows + k) * n + g));
    const float c2 = static_cast<float>(load_param<T>(coeffs, (1 * rows + k) * n + g));
    const float c3 = static_cast<float>(load_param<T>(coeffs, (2 * rows + k) * n + g));
    return t * (c1 + t * (c2 + t * c3));
}

// Shape part of the adjoint inputs of a Gaussian with dynamics at time t:
// scales, normalised quaternion (and 1/|q|), rotation, 3D covariance, opacity.
template <typename T>
__device__ __forceinline__ void shape_inputs(const Args& a, int64_t g, float t, AdjIn& P) {
    const int64_t n = a.n;
    float q[4];
    for (int k = 0; k < 3; ++k) {
        float ls = static_cast<float>(load_param<T>(a.log_scales, k * n + g));
        if (a.scale_coeffs) ls = ls + cubic_in_t<T>(a, a.scale_coeffs, 3, k, g, t);
        P.s[k] = expf(ls);
    }
    for (int k = 0; k < 4; ++k) {
        q[k] = static_cast<float>(load_param<T>(a.quats, k * n + g));
        if (a.quat_coeffs) q[k] = q[k] + cubic_in_t<T>(a, a.quat_coeffs, 4, k, g, t);
    }
    P.iqn = 1.0f / sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    for (int k = 0; k < 4; ++k) P.qh[k] = q[k] * P.iqn;
    const float eta = static_cast<float>(load_param<T>(a.opacity_logits, g));
    P.o = 1.0f / (1.0f + expf(-eta));
    {
        const float w = P.qh[0], x = P.qh[1], y = P.qh[2], z = P.qh[3];
        float* R = P.R;
        R[0] = 1.f - 2.f * (y * y + z * z); R[1] = 2.f * (x * y - w * z);       R[2] = 2.f * (x * z + w * y);
        R[3] = 2.f * (x * y + w * z);       R[4] = 1.f - 2.f * (x * x + z * z); R[5] = 2.f * (y * z - w * x);
        R[6] = 2.f * (x * z - w * y);       R[7] = 2.f * (y * z + w * x);       R[8] = 1.f - 2.f * (x * x + y * y);
    }
    {
        float M[9];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) M[i * 3 + j] = P.R[i * 3 + j] * P.s[j];
        P.Sig[0] = M[0] * M[0] + M[1] * M[1] + M[2] * M[2];
        P.Sig[1] = M[0] * M[3] + M[1] * M[4] + M[2] * M[5];
        P.Sig[2] = M[0] * M[6] + M[1] * M[7] + M[2] * M[8];
        P.Sig[3] = M[3] * M[3] + M[4] * M[4] + M[5] * M[5];
        P.Sig[4] = M[3] * M[6] + M[4] * M[7] + M[5] * M[8];
        P.Sig[5] = M[6] * M[6] + M[7] * M[7] + M[8] * M[8];
    }
}

// Without dynamics: the forward's frame-independent shape.
__device__ __forceinline__ void static_inputs(const Args& a, int64_t g, AdjIn& P) {
    for (int k = 0; k < 6; ++k) P.Sig[k] = static_cast<float>(a.shapes[g].Sig[k]);
    P.o = static_cast<float>(a.shapes[g].o);
}

// Camera-space position of the mean P.mu and the projection Jacobian times the
// camera rotation.
__device__ __forceinline__ void frame_geometry(const Args& a, const float* Rc, const float* tc, AdjIn& P) {
    for (int i = 0; i < 3; ++i)
        P.m[i] = tc[i] + Rc[i * 3 + 0] * P.mu[0] + Rc[i * 3 + 1] * P.mu[1] + Rc[i * 3 + 2] * P.mu[2];
    P.iz = 1.0f / P.m[2];
    const float iz = P.iz;
    const float j00 = a.fx * iz, j02 = -a.fx * P.m[0] * iz * iz;
    const float j11 = a.fy * iz, j12 = -a.fy * P.m[1] * iz * iz;
    for (int j = 0; j < 3; ++j) {
        P.T[j] = j00 * Rc[0 * 3 + j] + j02 * Rc[2 * 3 + j];
        P.T[3 + j] = j11 * Rc[1 * 3 + j] + j12 * Rc[2 * 3 + j];
    }
}

// Frame part: the mean at time t (B-spline, cubic or static), its camera-space
// position, the projection Jacobian times the camera rotation, and the conic
// of the forward record (the FP64 value rounded once: exactly the one the
// compositing kernels used).
template <bool DYN, typename T>
__device__ __forceinline__ void frame_inputs(const Args& a, int64_t g, const Record& rec, const float* Rc,
                                             const float* tc, float t, AdjIn& P) {
    const int64_t n = a.n;
    P.span = 0;
    if (DYN && a.n_ctrl > 0) {
        P.span = spline_basis<float>(a.n_ctrl, fminf(fmaxf(t, 0.0f), 1.0f), P.N);
        for (int k = 0; k < 3; ++k) {
            float mu = 0.0f;
            for (int r = 0; r < 4; ++r)
                if (P.N[r] != 0.0f)
                    mu += P.N[r] * static_cast<float>(
                                       load_param<T>(a.ctrl, (static_cast<int64_t>(P.span + r) * 3 + k) * n + g));
            P.mu[k] = mu;
        }
    } else {
        for (int k = 0; k < 3; ++k) {
            float mu = static_cast<float>(load_param<T>(a.means, k * n + g));
            if (a.mean_coeffs) mu = mu + cubic_in_t<T>(a, a.mean_coeffs, 3, k, g, t);
            P.mu[k] = mu;
        }
    }
    frame_geometry(a, Rc, tc, P);
    P.A[0] = rec.a;
    P.A[1] = rec.b;
    P.A[2] = rec.c;
}

// dL/dSig (symmetric, stored xx xy xz yy yz zz) -> gradients of the stored
// log-scales (out 0-2) and the unnormalised quaternion (out 3-6), through
// Sig = M M^T, M = R diag(s): dM = 2 G M, dR = dM diag(s), ds_j = sum_i dM_ij R_ij.
// The quaternion's sums cancel (for equal scales they vanish), which amplifies
// rounding: Gaussians without dynamics, which take this once after the sum
// over frames, take it in FP64.
template <typename F, typename Shape>
__device__ __forceinline__ void sigma_adjoint(const F G[6], const Shape& P, F out[7]) {
    const F Gm[9] = {G[0], G[1], G[2], G[1], G[3], G[4], G[2], G[4], G[5]};
    F ds[3] = {F(0), F(0), F(0)};
    F gq[4] = {F(0), F(0), F(0), F(0)};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const F V = Gm[i * 3 + 0] * P.R[0 * 3 + j] + Gm[i * 3 + 1] * P.R[1 * 3 + j] +
                        Gm[i * 3 + 2] * P.R[2 * 3 + j];
            const F dM = F(2) * P.s[j] * V;
            ds[j] += dM * P.R[i * 3 + j];
            add_rot_partial<F>(i * 3 + j, dM * P.s[j], P.qh, gq);
        }
    for (int k = 0; k < 3; ++k) out[k] = ds[k] * P.s[k];
    // q_hat = q / |q|
    const F dot = P.qh[0] * gq[0] + P.qh[1] * gq[1] + P.qh[2] * gq[2] + P.qh[3] * gq[3];
    for (int k = 0; k < 4; ++k) out[3 + k] = (gq[k] - P.qh[k] * dot) * P.iqn;
}

// The FP64 shape sigma_adjoint takes for Gaussians without dynamics.
struct ShapeAdj {
    double s[3], qh[4], iqn, R[9];
};

template <typename T>
__device__ __forceinline__ void shape_f64(const Args& a, int64_t g, ShapeAdj& P) {
    const int64_t n = a.n;
    double q[4];
    for (int k = 0; k < 3; ++k) P.s[k] = exp(load_param<T>(a.log_scales, k * n + g));
    for (int k = 0; k < 4; ++k) q[k] = load_param<T>(a.quats, k * n + g);
    P.iqn = 1.0 / sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    for (int k = 0; k < 4; ++k) P.qh[k] = q[k] * P.iqn;
    rot_from_quat(P.qh[0], P.qh[1], P.qh[2], P.qh[3], P.R);
}

// dL/dSig summed over the frames to log-scales and quaternion.  A Gaussian
// culled in every frame (e.g. for non-finite parameters) has dL/dSig = 0
// exactly; its shape may hold NaN, so it is not taken through the chain (0 * NaN
// would poison its gradient).
template <typename T>
__device__ __forceinline__ void static_shape_adjoint(const Args& a, int64_t g, const double* Gs, double out[7]) {
    bool touched = false;
    for (int k = 0; k < 6; ++k) touched = touched || Gs[k] != 0.0;
    for (int k = 0; k < 7; ++k) out[k] = 0.0;
    if (!touched) return;
    ShapeAdj S;
    shape_f64<T>(a, g, S);
    sigma_adjoint<double>(Gs, S, out);
}

// Chain rule for one (frame, Gaussian).  d: dL/d(u, v, A00, A01, A11, o, r, g,
// b) with A01 the single off-diagonal conic parameter (it enters q twice).
// Writes the gradients w.r.t. the frame's parameter values to gout (mean 0-2,
// log-scales 3-5, quaternion 6-9, opacity logit 10, colour 11-13; with
// SIGMA_OUT, dL/dSig at 3-8 instead of 3-9) and adds the pose gradient
// (dL/dRc row-major 0-8, dL/dtc 9-11) to pose.
template <bool SIGMA_OUT>
__device__ __forceinline__ void projection_adjoint(const Args& a, const float* Rc, const AdjIn& P,
                                                   const float d[9], float gout[14], float (&pose)[12],
                                                   float gintr[4]) {
    const float A0 = P.A[0], A1 = P.A[1], A2 = P.A[2];
    // gradient w.r.t. the symmetric conic matrix
    const float G00 = d[2], G01 = 0.5f * d[3], G11 = d[4];
    // A = cov^-1  =>  dL/dcov = -A G A
    const float AG00 = A0 * G00 + A1 * G01, AG01 = A0 * G01 + A1 * G11;
    const float AG10 = A1 * G00 + A2 * G01, AG11 = A1 * G01 + A2 * G11;
    const float C00 = -(AG00 * A0 + AG01 * A1);
    const float C01 = -0.5f * ((AG00 * A1 + AG01 * A2) + (AG10 * A0 + AG11 * A1));
    const float C11 = -(AG10 * A1 + AG11 * A2);
    // cov = T Sig T^T + dil I with T = J Rc (2x3); CT = C T
    const float* Tm = P.T;
    float CT[6];
    for (int j = 0; j < 3; ++j) {
        CT[j] = C00 * Tm[j] + C01 * Tm[3 + j];
        CT[3 + j] = C01 * Tm[j] + C11 * Tm[3 + j];
    }
    // dT = 2 C T Sig  (Sig symmetric, stored xx xy xz yy yz zz)
    const float* S = P.Sig;
    float dT[6];
    for (int i = 0; i < 2; ++i) {
        const float c0 = CT[i * 3 + 0], c1 = CT[i * 3 + 1], c2 = CT[i * 3 + 2];
        dT[i * 3 + 0] = 2.0f * (c0 * S[0] + c1 * S[1] + c2 * S[2]);
        dT[i * 3 + 1] = 2.0f * (c0 * S[1] + c1 * S[3] + c2 * S[4]);
        dT[i * 3 + 2] = 2.0f * (c0 * S[2] + c1 * S[4] + c2 * S[5]);
    }
    // T = J Rc with J = [[j00, 0, j02], [0, j11, j12]]
    const float mx = P.m[0], my = P.m[1];
    const float iz = P.iz, iz2 = iz * iz, iz3 = iz2 * iz;
    const float fx = a.fx, fy = a.fy;
    const float j00 = fx * iz, j02 = -fx * mx * iz2, j11 = fy * iz, j12 = -fy * my * iz2;
    float dJ00 = 0.f, dJ02 = 0.f, dJ11 = 0.f, dJ12 = 0.f;
    for (int j = 0; j < 3; ++j) {
        dJ00 += dT[j] * Rc[0 * 3 + j];
        dJ02 += dT[j] * Rc[2 * 3 + j];
        dJ11 += dT[3 + j] * Rc[1 * 3 + j];
        dJ12 += dT[3 + j] * Rc[2 * 3 + j];
        pose[0 * 3 + j] += j00 * dT[j];
        pose[1 * 3 + j] += j11 * dT[3 + j];
        pose[2 * 3 + j] += j02 * dT[j] + j12 * dT[3 + j];
    }
    // intrinsics: u = fx mx/mz + cx, v = fy my/mz + cy, J00 = fx/mz,
    // J02 = -fx mx/mz^2, J11 = fy/mz, J12 = -fy my/mz^2
    gintr[0] = d[0] * mx * iz + dJ00 * iz - dJ02 * mx * iz2;
    gintr[1] = d[1] * my * iz + dJ11 * iz - dJ12 * my * iz2;
    gintr[2] = d[0];
    gintr[3] = d[1];
    // J(m) and (u, v)(m)
    float dm[3];
    dm[0] = -dJ02 * fx * iz2 + d[0] * fx * iz;
    dm[1] = -dJ12 * fy * iz2 + d[1] * fy * iz;
    dm[2] = -dJ00 * fx * iz2 + dJ02 * 2.0f * fx * mx * iz3 - dJ11 * fy * iz2 + dJ12 * 2.0f * fy * my * iz3 -
            d[0] * fx * mx * iz2 - d[1] * fy * my * iz2;
    // m = Rc mu + tc
    for (int k = 0; k < 3; ++k) {
        gout[k] = Rc[0 * 3 + k] * dm[0] + Rc[1 * 3 + k] * dm[1] + Rc[2 * 3 + k] * dm[2];
        pose[9 + k] += dm[k];
    }
    for (int i = 0; i < 3; ++i)
        for (int k = 0; k < 3; ++k) pose[i * 3 + k] += dm[i] * P.mu[k];
    // dL/dSig = T^T C T; static Gaussians return it (summed over frames and
    // taken through sigma_adjoint once), the others apply sigma_adjoint per frame
    float G[6];
    G[0] = Tm[0] * CT[0] + Tm[3] * CT[3];
    G[1] = Tm[0] * CT[1] + Tm[3] * CT[4];
    G[2] = Tm[0] * CT[2] + Tm[3] * CT[5];
    G[3] = Tm[1] * CT[1] + Tm[4] * CT[4];
    G[4] = Tm[1] * CT[2] + Tm[4] * CT[5];
    G[5] = Tm[2] * CT[2] + Tm[5] * CT[5];
    if (SIGMA_OUT) {
        for (int k = 0; k < 6; ++k) gout[3 + k] = G[k];
        gout[9] = 0.0f;
    } else {
        sigma_adjoint<float>(G, P, gout + 3);
    }
    gout[10] = d[5] * P.o * (1.0f - P.o);
    gout[11] = d[6];
    gout[12] = d[7];
    gout[13] = d[8];
}

// Accumulator slots (FP64, in LDS) of the projection adjoint kernel.  The
// static layout holds the per-frame gradients of the mean (0-2), dL/dSig
// (3-8; slot 9 unused), opacity (10) and colour (11-13), and the cubic mean
// coefficients 14-22.  The dynamic layout (B-spline means and/or polynomial
// log-scales and quaternions, Eq. 2-3) holds the 14 at 0-13, a window of four
// control points 14-25 (point span + r, axis k at 14 + 3 r + k) or, as the two
// exclude each other, the cubic mean coefficients 14-22, the log-scale
// coefficients 26-34 and the quaternion coefficients 35-46.
template <bool DYN>
struct AccLayout {
    static constexpr int N = DYN ? 47 : 23;
    static constexpr int CUBIC = 14, WIN = 14, SCALE = 26, QUAT = 35;
};

// View-dependent colour (SH, Sec. 3.1): given dL/d(colour) of one frame,
// add Y_k(d) dL/dc to the coefficient accumulators and return, through the
// unit direction d = v / |v|, v = mu - C, dL/dv (it adds to dL/dmu, and
// -dL/dv is the gradient of the camera centre C = -Rc^T tc).
template <int NT, typename T>
__device__ __forceinline__ void sh_adjoint(const Args& a, int64_t g, const AdjIn& P, const float* camC,
                                           const float dc[3], float (*acc_sh)[NT], int tid, float dv[3]) {
    const int64_t n = a.n;
    float v[3];
    for (int i = 0; i < 3; ++i) v[i] = P.mu[i] - camC[i];
    const float vn = sqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const float iv = vn > 0.0f ? 1.0f / vn : 0.0f;
    const float d[3] = {v[0] * iv, v[1] * iv, v[2] * iv};
    float Y[15], G[15][3];
    sh_eval<float>(3, d[0], d[1], d[2], Y, G);  // all degrees (static indexing); unused ones are skipped
    const int nb = sh_count(a.sh_degree);
    float dd[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 15; ++k) {  // static indices keep Y and G in registers
        if (k < nb) {
            float w = 0.f;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                acc_sh[k * 3 + c][tid] += Y[k] * dc[c];
                w += dc[c] * static_cast<float>(load_param<T>(a.sh, (static_cast<int64_t>(k) * 3 + c) * n + g));
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) dd[j] += w * G[k][j];
        }
    }
    const float dot = d[0] * dd[0] + d[1] * dd[1] + d[2] * dd[2];
    for (int j = 0; j < 3; ++j) dv[j] = (dd[j] - d[j] * dot) * iv;
}

// Sum of a Gaussian's marked partial records in one frame (cnt slots from base
// on), in slot order in FP64, rounded once.  PU records per round, their loads
// issued together with the marks (past the end they repeat a valid record and
// are not added; records the adjoint did not write this pass hold stale values
// and are not added either).
template <uint32_t PU>
struct PartialRound {
    float r[PU][PART];
    uint32_t w0, w1;  // words holding the round's marks
    __device__ __forceinline__ void load(const Args& a, uint32_t base, uint32_t cnt, uint32_t k0) {
        const uint32_t wi = (base + k0) >> 5;
        w0 = a.pused[wi];
        w1 = a.pused[wi + 1];
#pragma unroll
        for (uint32_t u = 0; u < PU; ++u) {
            const uint32_t k = k0 + u < cnt ? k0 + u : k0;
            const float* pp = a.part + static_cast<int64_t>(base + k) * PART;
#pragma unroll
            for (int m = 0; m < PART; ++m) r[u][m] = pp[m];
        }
    }
    __device__ __forceinline__ void add(uint32_t base, uint32_t cnt, uint32_t k0, double (&s)[PART]) const {
        const uint32_t bits = static_cast<uint32_t>(((static_cast<uint64_t>(w1) << 32) | w0) >> ((base + k0) & 31u));
#pragma unroll
        for (uint32_t u = 0; u < PU; ++u)
            if (k0 + u < cnt && ((bits >> u) & 1u))
#pragma unroll
                for (int m = 0; m < PART; ++m) s[m] += r[u][m];
    }
};
constexpr uint32_t PU = 4;

// dL/dSig (xx xy xz yy yz zz) of one (frame, Gaussian) in FP64: from the sums s
// of its partial records and the conic A through dL/dcov = -A G A and T^T C T.
// In FP32 the rounding of the conic's and T's products, amplified by a needle's
// axis ratio, was most of the quaternion gradient's error: 1.3e-6 of its norm
// on one 960x540 frame of 100k Gaussians, 0.25e-6 so (medians of 20 scenes).
__device__ __forceinline__ void sigma_gradient_f64(const Args& a, const double* Rc, const double* tc,
                                                   const float mu[3], const float A[3], const double s[PART],
                                                   double G[6]) {
    double m[3], T[6];
    for (int i = 0; i < 3; ++i) m[i] = tc[i] + Rc[i * 3 + 0] * mu[0] + Rc[i * 3 + 1] * mu[1] + Rc[i * 3 + 2] * mu[2];
    const double iz = 1.0 / m[2];
    const double j00 = a.fx * iz, j02 = -a.fx * m[0] * iz * iz;
    const double j11 = a.fy * iz, j12 = -a.fy * m[1] * iz * iz;
    for (int j = 0; j < 3; ++j) {
        T[j] = j00 * Rc[0 * 3 + j] + j02 * Rc[2 * 3 + j];
        T[3 + j] = j11 * Rc[1 * 3 + j] + j12 * Rc[2 * 3 + j];
    }
    const double A0 = A[0], A1 = A[1], A2 = A[2];
    const double G00 = s[2], G01 = 0.5 * s[3], G11 = s[4];
    const double AG00 = A0 * G00 + A1 * G01, AG01 = A0 * G01 + A1 * G11;
    const double AG10 = A1 * G00 + A2 * G01, AG11 = A1 * G01 + A2 * G11;
    const double C00 = -(AG00 * A0 + AG01 * A1);
    const double C01 = -0.5 * ((AG00 * A1 + AG01 * A2) + (AG10 * A0 + AG11 * A1));
    const double C11 = -(AG10 * A1 + AG11 * A2);
    double CT[6];
    for (int j = 0; j < 3; ++j) {
        CT[j] = C00 * T[j] + C01 * T[3 + j];
        CT[3 + j] = C01 * T[j] + C11 * T[3 + j];
    }
    G[0] = T[0] * CT[0] + T[3] * CT[3];
    G[1] = T[0] * CT[1] + T[3] * CT[4];
    G[2] = T[0] * CT[2] + T[3] * CT[5];
    G[3] = T[1] * CT[1] + T[4] * CT[4];
    G[4] = T[1] * CT[2] + T[4] * CT[5];
    G[5] = T[2] * CT[2] + T[5] * CT[5];
}

// The adjoint of Gaussians without dynamics or SH: one lane per Gaussian and
// SPLIT waves per 64 Gaussians, each taking a contiguous part of the frames
// (quarters rather than halves shorten the last round of workgroups, which runs
// almost alone); the parts' FP64 sums are added in order at the end.  Fewer than
// four frames take SPLIT = 1, which leaves no wave of a workgroup idle: the
// adjoint of one 960x540 frame of 100k Gaussians 48 -> 26 us.
//
// Bound by the latency and the rate of the record reads (36 bytes each, in runs
// of a few).  Rounds of four records and sums in registers hold it at three
// waves per SIMD where rounds of eight with the sums in LDS held two; the next
// frame's count, offset and conic are requested after this frame's first
// records, not before, so that waiting for the records does not wait for them:
// 544 -> 526 us on the 50-frame 960x540 clip, 1,869 -> 1,648 us on the 32-frame
// 1080p clip with cubic means.  (Staging a wave's records through LDS in
// coalesced reads cut the loads to a quarter but took twice the VALU: 613 us.)
//
// LARGE: for up to three frames of Gaussians of many tiles (large_gaussians), a
// wave per frame and, after the first, rounds of eight records, which halve the
// chain of a lane's dependent rounds but leave two waves per SIMD: two 960x540
// frames of 20k Gaussians of 29 tiles 97 -> 60 us, three 139 -> 64; of 200k of four
// tiles 47 and 59 us with rounds of four in one wave, 55 and 80 so.
template <int SPLIT, bool CUBIC, typename T, bool LARGE>
__global__ __launch_bounds__(64 * SPLIT) void k_adjoint_static(Args a) {
    if (overflowed(a.status)) return;
    constexpr int FC = 16;  // frames whose cameras and pose sums are in LDS
    constexpr int NA = CUBIC ? 23 : 14;
    // FP64 for dL/dSig where a few frames do not average its rounding out.  Over
    // twelve frames it changes the quaternion gradient's error by 3 % (median of
    // 30 scenes), and with cubic means its registers would leave two waves per
    // SIMD (1080p clip 1,641 -> 1,815 us).
    constexpr bool SIGMA_F64 = SPLIT < 4;
    __shared__ double camd[SIGMA_F64 ? SPLIT : 1][SIGMA_F64 ? FC : 1][12];
    __shared__ float cam[SPLIT][FC][12], wpose[SPLIT][FC][12];
    __shared__ double red[SPLIT][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int h = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n = a.n, g0 = static_cast<int64_t>(blockIdx.x) * 64;
    const int64_t g = g0 + lane;
    const bool live = g < n;
    const int64_t gs = live ? g : n - 1;
    const int fpart = (a.frames + SPLIT - 1) / SPLIT;
    const int fb = min(h * fpart, a.frames), fe = min(fb + fpart, a.frames);

    AdjIn P = {};
    float mu0[3], mc[9];
    for (int k = 0; k < 3; ++k) mu0[k] = static_cast<float>(load_param<T>(a.means, k * n + gs));
    if (CUBIC)
        for (int k = 0; k < 9; ++k) mc[k] = static_cast<float>(load_param<T>(a.mean_coeffs, k * n + gs));
    static_inputs(a, gs, P);

    double acc[NA], iacc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < NA; ++k) acc[k] = 0.0;

    uint32_t cnt1 = 0u, base1 = 0u;  // of the frame about to be taken
    float4 rec1 = {};
    auto slots = [&](int f, uint32_t& c, uint32_t& b) {
        const int64_t i = static_cast<int64_t>(f) * n + gs;
        c = live ? a.gcnt[i] : 0u;
        b = a.goff[i];
    };
    auto conic = [&](int f) {
        return *reinterpret_cast<const float4*>(&a.rec[static_cast<int64_t>(f) * n + gs].a);
    };
    auto prefetch = [&](int f) {
        if (f >= fe) return;
        slots(f, cnt1, base1);
        rec1 = conic(f);
    };
    prefetch(fb);
#pragma unroll 1
    for (int c0 = 0; c0 < fpart; c0 += FC) {  // the same chunk count in every wave (uniform barriers)
        const int f0 = fb + c0;
        const int nf = max(0, min(fe - f0, FC));
        __syncthreads();  // the previous chunk's cameras and pose sums are consumed
        for (int q = tid; q < SPLIT * FC; q += 64 * SPLIT) {
            const int hh = q / FC, fi = q % FC;
            const int ff = hh * fpart + c0 + fi;
            if (ff < min((hh + 1) * fpart, a.frames)) {
                const CamD c = load_camera(a.poses + 7 * ff);
                if (SIGMA_F64) {
                    for (int k = 0; k < 9; ++k) camd[hh][fi][k] = c.ok ? c.R[k] : 0.0;
                    for (int k = 0; k < 3; ++k) camd[hh][fi][9 + k] = c.ok ? c.t[k] : 0.0;
                }
                for (int k = 0; k < 9; ++k) cam[hh][fi][k] = c.ok ? static_cast<float>(c.R[k]) : 0.0f;
                for (int k = 0; k < 3; ++k) cam[hh][fi][9 + k] = c.ok ? static_cast<float>(c.t[k]) : 0.0f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int fi = 0; fi < nf; ++fi) {
            const int f = f0 + fi;
            uint32_t cnt = cnt1;
            const uint32_t base = base1;
            const float4 rec = rec1;
            if (static_cast<int64_t>(base) + cnt > a.k_cap) cnt = 0u;  // only after an internal error
            const float* camR = cam[h][fi];
            const float* camT = cam[h][fi] + 9;
            float pose[12];
            for (int k = 0; k < 12; ++k) pose[k] = 0.0f;
            if (cnt) {
                PartialRound<PU> R;  // requested before the frame's geometry, which does not need it
                R.load(a, base, cnt, 0u);
                prefetch(f + 1);
                const float t = a.times ? a.times[f] : a.t0;
                for (int k = 0; k < 3; ++k) {
                    P.mu[k] = mu0[k];
                    if (CUBIC) P.mu[k] = mu0[k] + t * (mc[k] + t * (mc[3 + k] + t * mc[6 + k]));
                }
                frame_geometry(a, camR, camT, P);
                P.A[0] = rec.x;
                P.A[1] = rec.y;
                P.A[2] = rec.z;
                double s[PART] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
                if constexpr (LARGE) {
                    R.add(base, cnt, 0u, s);
#pragma unroll 1
                    for (uint32_t k0 = PU; k0 < cnt; k0 += 8) {
                        PartialRound<8> M;
                        M.load(a, base, cnt, k0);
                        M.add(base, cnt, k0, s);
                    }
                } else {
                    for (uint32_t k0 = 0;;) {
                        R.add(base, cnt, k0, s);
                        k0 += PU;
                        if (k0 >= cnt) break;
                        R.load(a, base, cnt, k0);
                    }
                }
                float d[PART];
                for (int k = 0; k < PART; ++k) d[k] = static_cast<float>(s[k]);
                float go[14], gi[4];
                projection_adjoint<true>(a, camR, P, d, go, pose, gi);
                for (int k = 0; k < 4; ++k) iacc[k] += gi[k];
                if (SIGMA_F64) {
                    double G[6];
                    sigma_gradient_f64(a, camd[h][fi], camd[h][fi] + 9, P.mu, P.A, s, G);
                    for (int k = 0; k < 6; ++k) {
                        acc[3 + k] += G[k];
                        go[3 + k] = 0.0f;
                    }
                }
                for (int k = 0; k < 14; ++k) acc[k] += go[k];
                if (CUBIC) {
                    const double t1 = t, t2 = t1 * t1, t3 = t2 * t1;
                    for (int k = 0; k < 3; ++k) {
                        acc[14 + k] += go[k] * t1;
                        acc[17 + k] += go[k] * t2;
                        acc[20 + k] += go[k] * t3;
                    }
                }
            }
            else prefetch(f + 1);
            if (a.g_poses) {  // wave sums of this frame's pose contributions
                float v[16];
#pragma unroll
                for (int k = 0; k < 12; ++k) v[k] = pose[k];
#pragma unroll
                for (int k = 12; k < 16; ++k) v[k] = 0.0f;
                const float x = reduce_scatter16(v, lane);
                const int idx = reduce_scatter16_index(lane);
                if ((lane & 3) == 0 && idx < 12) wpose[h][fi][idx] = x;
            }
        }
        if (a.g_poses) {
            __syncthreads();
            for (int q = tid; q < SPLIT * FC * 12; q += 64 * SPLIT) {
                const int hh = q / (FC * 12), r = q % (FC * 12), fi = r / 12, k = r % 12;
                const int ff = hh * fpart + c0 + fi;
                if (ff < min((hh + 1) * fpart, a.frames))
                    a.pose_part[(static_cast<int64_t>(blockIdx.x) * a.frames + ff) * 12 + k] =
                        static_cast<double>(wpose[hh][fi][k]);
            }
        }
    }
    if (a.g_intr) {
        for (int k = 0; k < 4; ++k) {
            const double v = wave_sum_f64(iacc[k]);
            if (lane == 0) red[h][k] = v;
        }
        __syncthreads();
        if (tid < 4) {
            double v = 0.0;
            for (int hh = 0; hh < SPLIT; ++hh) v += red[hh][tid];
            a.intr_part[static_cast<int64_t>(blockIdx.x) * 4 + tid] = v;
        }
    }
    if (SPLIT > 1) {  // add the later parts' sums to part 0's, in order
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            __syncthreads();
            red[h][lane] = acc[k];
            __syncthreads();
            if (h == 0)
                for (int hh = 1; hh < SPLIT; ++hh) acc[k] += red[hh][lane];
        }
    }
    if (!live || h != 0) return;
    auto put = [&](float* dst, int64_t idx, double v) {
        if (!dst) return;
        if (a.accumulate) dst[idx] += static_cast<float>(v);
        else dst[idx] = static_cast<float>(v);
    };
    double gsq[7];
    static_shape_adjoint<T>(a, g, acc + 3, gsq);
    for (int k = 0; k < 3; ++k) {
        put(a.g_means, k * n + g, acc[k]);
        put(a.g_log_scales, k * n + g, gsq[k]);
        put(a.g_colors, k * n + g, acc[11 + k]);
    }
    for (int k = 0; k < 4; ++k) put(a.g_quats, k * n + g, gsq[3 + k]);
    put(a.g_opacity, g, acc[10]);
    if (CUBIC)
        for (int k = 0; k < 9; ++k) put(a.g_coeffs, k * n + g, acc[14 + k]);
}

// ---------------------------------------------------------------------------
// The adjoint with dynamics or SH, or of large Gaussians, in two kernels.  One lane per (frame,
// Gaussian) takes the chain rule down to the frame's parameter values and
// stores them (k_adjoint_frames); one lane per Gaussian then sums them over the
// frames in FP64 with the frames' weights (k_adjoint_sum).  In one kernel, the
// frame's chain rule and up to 47 FP64 sums (and 45 SH sums) a lane held the
// chip at one wave per SIMD, waiting on a Gaussian's records frame after frame:
// on the 50-frame 960x540 clip of 200k Gaussians 2,180 us with B-spline
// means and cubic covariance, 1,035 us so; 1,430 -> 822 us with SH of degree 3.
// (Without either, one kernel with its 14 sums in registers is faster, 519 us
// against 703, and 1,634 against 2,096 us on the 1080p clip, unless Gaussians are
// large and few, see large_gaussians.)  The stored values cost twice their 52 to
// 68 bytes per (frame, Gaussian); they lie in the sort's key buffers, which
// nothing reads after the sort.  Where those are too small (less than 1.625
// intersections of capacity per (frame, Gaussian) with SH, 1.75 with dynamics,
// 2.125 with both) the one-kernel form below runs.
// ---------------------------------------------------------------------------
template <bool DYN, bool SH>
constexpr int frame_values() { return (DYN ? 14 : 13) + (DYN && SH ? 3 : 0); }

struct FrameStore {
    float *lo, *hi;     // frames [0, lo_frames) and the rest
    int lo_frames;
    int64_t stride;     // floats per frame
    double* intr;       // [frame][block][4] intrinsics partials
    int blocks;         // workgroups per frame of k_adjoint_frames
    __device__ __forceinline__ float* frame(int f) const {
        return f < lo_frames ? lo + f * stride : hi + (f - lo_frames) * stride;
    }
};

// dL/dv of the view-dependent colour (see sh_adjoint) and the unit direction.
template <typename T>
__device__ __forceinline__ void sh_direction_adjoint(const Args& a, int64_t g, const float mu[3], const float* camC,
                                                     const float dc[3], float d[3], float dv[3]) {
    const int64_t n = a.n;
    float v[3];
    for (int i = 0; i < 3; ++i) v[i] = mu[i] - camC[i];
    const float vn = sqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const float iv = vn > 0.0f ? 1.0f / vn : 0.0f;
    for (int i = 0; i < 3; ++i) d[i] = v[i] * iv;
    float Y[15], G[15][3];
    sh_eval<float>(3, d[0], d[1], d[2], Y, G);
    float dd[3] = {0.f, 0.f, 0.f};
    // every degree, with no branch between the loads; the terms past the
    // scene's degree repeat its last coefficients and weigh nothing
    const int nb = sh_count(a.sh_degree);
#pragma unroll
    for (int k = 0; k < 15; ++k) {
        const int kk = k < nb ? k : nb - 1;
        float w = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            w += dc[c] * static_cast<float>(load_param<T>(a.sh, (static_cast<int64_t>(kk) * 3 + c) * n + g));
        w = k < nb ? w : 0.0f;
#pragma unroll
        for (int j = 0; j < 3; ++j) dd[j] += w * G[k][j];
    }
    const float dot = d[0] * dd[0] + d[1] * dd[1] + d[2] * dd[2];
    for (int j = 0; j < 3; ++j) dv[j] = (dd[j] - d[j] * dot) * iv;
}

template <bool DYN, bool SH, typename T>
__global__ __launch_bounds__(256) void k_adjoint_frames(Args a, FrameStore store) {
    if (overflowed(a.status)) return;
    int block, f;
    if (!block_and_frame(store.blocks, a.frames, block, f)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t n = a.n, g = static_cast<int64_t>(block) * 256 + tid;
    __shared__ float cam[15];  // R, t, centre
    __shared__ float weights[4];
    __shared__ int span;
    __shared__ float wpose[4][12], gintr[4][256];
    const float t = a.times ? a.times[f] : a.t0;
    uint32_t cnt = 0u, base = 0u;
    if (g < n) {
        const int64_t i = static_cast<int64_t>(f) * n + g;
        cnt = a.gcnt[i];
        base = a.goff[i];
        if (static_cast<int64_t>(base) + cnt > a.k_cap) cnt = 0u;  // only after an internal error
    }
    if (tid == 0) {
        const CamD c = load_camera(a.poses + 7 * f);
        for (int k = 0; k < 9; ++k) cam[k] = c.ok ? static_cast<float>(c.R[k]) : 0.0f;
        for (int k = 0; k < 3; ++k) cam[9 + k] = c.ok ? static_cast<float>(c.t[k]) : 0.0f;
        for (int i = 0; i < 3; ++i)
            cam[12 + i] = c.ok ? static_cast<float>(-(c.R[0 * 3 + i] * c.t[0] + c.R[1 * 3 + i] * c.t[1] +
                                                      c.R[2 * 3 + i] * c.t[2]))
                               : 0.0f;
    }
    if (DYN && a.n_ctrl > 0 && tid == 64) {
        float N[4];
        span = spline_basis<float>(a.n_ctrl, fminf(fmaxf(t, 0.0f), 1.0f), N);
        for (int r = 0; r < 4; ++r) weights[r] = N[r];
    }
    __syncthreads();
    float pose[12], gi[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < 12; ++k) pose[k] = 0.0f;
    if (cnt) {
        PartialRound<PU> R;
        R.load(a, base, cnt, 0u);
        const float4 rec = *reinterpret_cast<const float4*>(&a.rec[static_cast<int64_t>(f) * n + g].a);
        AdjIn P = {};
        if (DYN) {
            shape_inputs<T>(a, g, t, P);
        } else {
            static_inputs(a, g, P);
        }
        for (int k = 0; k < 3; ++k) {
            float mu = 0.0f;
            if (DYN && a.n_ctrl > 0) {
                for (int r = 0; r < 4; ++r)
                    if (weights[r] != 0.0f)
                        mu += weights[r] * static_cast<float>(
                                               load_param<T>(a.ctrl, (static_cast<int64_t>(span + r) * 3 + k) * n + g));
            } else {
                mu = static_cast<float>(load_param<T>(a.means, k * n + g));
                if (a.mean_coeffs) mu = mu + cubic_in_t<T>(a, a.mean_coeffs, 3, k, g, t);
            }
            P.mu[k] = mu;
        }
        frame_geometry(a, cam, cam + 9, P);
        P.A[0] = rec.x;
        P.A[1] = rec.y;
        P.A[2] = rec.z;
        double s[PART] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (uint32_t k0 = 0;;) {
            R.add(base, cnt, k0, s);
            k0 += PU;
            if (k0 >= cnt) break;
            R.load(a, base, cnt, k0);
        }
        float d[PART];
        for (int k = 0; k < PART; ++k) d[k] = static_cast<float>(s[k]);
        float go[14];
        projection_adjoint<!DYN>(a, cam, P, d, go, pose, gi);
        float* out = store.frame(f) + g;
        if (SH) {
            const float dc[3] = {go[11], go[12], go[13]};
            float dir[3], dv[3];
            sh_direction_adjoint<T>(a, g, P.mu, cam + 12, dc, dir, dv);
            for (int j = 0; j < 3; ++j) {
                go[j] += dv[j];
                // C = -Rc^T tc, dL/dC = -dv: dL/dtc = Rc dv, dL/dRc[j][i] = tc[j] dv[i]
                pose[9 + j] += cam[j * 3 + 0] * dv[0] + cam[j * 3 + 1] * dv[1] + cam[j * 3 + 2] * dv[2];
                for (int i = 0; i < 3; ++i) pose[j * 3 + i] += cam[9 + j] * dv[i];
                if (DYN) out[(14 + j) * n] = dir[j];
            }
        }
        for (int k = 0; k < (DYN ? 14 : 9); ++k) out[k * n] = go[k];
        if (!DYN)
            for (int k = 9; k < 13; ++k) out[k * n] = go[k + 1];
    }
    float v[16];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = pose[k];
#pragma unroll
    for (int k = 12; k < 16; ++k) v[k] = 0.0f;
    const float x = reduce_scatter16(v, lane);
    const int idx = reduce_scatter16_index(lane);
    if ((lane & 3) == 0 && idx < 12) wpose[w][idx] = x;
    for (int k = 0; k < 4; ++k) gintr[k][tid] = gi[k];
    __syncthreads();
    if (tid < 12) {
        double sum = 0.0;
        for (int ww = 0; ww < 4; ++ww) sum += static_cast<double>(wpose[ww][tid]);
        a.pose_part[(static_cast<int64_t>(block) * a.frames + f) * 12 + tid] = sum;
    }
    // wave w sums intrinsics gradient w in FP64
    double sum = 0.0;
    for (int q = 0; q < 4; ++q) sum += static_cast<double>(gintr[w][lane + 64 * q]);
    sum = wave_sum_f64(sum);
    if (lane == 0) store.intr[(static_cast<int64_t>(f) * store.blocks + block) * 4 + w] = sum;
}

// Sums the stored values over the frames.
template <bool DYN, bool SH, typename T>
__global__ __launch_bounds__(128) void k_adjoint_sum(Args a, FrameStore store) {
    if (overflowed(a.status)) return;
    constexpr int NV = frame_values<DYN, SH>();
    constexpr int FC = 64;
    __shared__ float ft[FC], weights[FC][4], centre[FC][3];
    __shared__ int spans[FC];
    const int tid = threadIdx.x;
    const int64_t n = a.n, g = static_cast<int64_t>(blockIdx.x) * 128 + tid;
    const bool live = g < n;
    const int64_t gs = live ? g : n - 1;
    const bool spline = DYN && a.n_ctrl > 0;
    const bool ctrl_out = spline && a.g_ctrl != nullptr;
    double acc[14], win_acc[DYN ? 12 : 1], sc[DYN ? 9 : 1], qc[DYN ? 12 : 1], cubic[DYN ? 1 : 9], sh[SH ? 45 : 1];
    for (int k = 0; k < 14; ++k) acc[k] = 0.0;
    for (double& v : win_acc) v = 0.0;
    for (double& v : sc) v = 0.0;
    for (double& v : qc) v = 0.0;
    for (double& v : cubic) v = 0.0;
    for (double& v : sh) v = 0.0;
    float mu0[3] = {0.f, 0.f, 0.f}, mc[9];
    if (SH && !DYN) {
        for (int k = 0; k < 3; ++k) mu0[k] = static_cast<float>(load_param<T>(a.means, k * n + gs));
        for (int k = 0; k < 9; ++k)
            mc[k] = a.mean_coeffs ? static_cast<float>(load_param<T>(a.mean_coeffs, k * n + gs)) : 0.0f;
    }
    // control-point window: sums of points win .. win + 3, flushed to memory
    // (added) when a frame falls in another knot span; cubic means, which
    // exclude control points, take its place
    int win = -1;
    auto flush_window = [&]() {
        if (win < 0 || !live) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                a.g_ctrl[(static_cast<int64_t>(win + r) * 3 + k) * n + g] += static_cast<float>(win_acc[(3 * r + k) % (DYN ? 12 : 1)]);
                win_acc[(3 * r + k) % (DYN ? 12 : 1)] = 0.0;
            }
    };
    if (ctrl_out && live && !a.accumulate)
        for (int64_t i = 0; i < static_cast<int64_t>(a.n_ctrl) * 3; ++i) a.g_ctrl[i * n + g] = 0.0f;
    float nv[NV];  // the next frame's values
    uint32_t ncnt = 0u;
    auto fetch = [&](int f) {
        ncnt = live ? a.gcnt[static_cast<int64_t>(f) * n + g] : 0u;
        const float* src = store.frame(f) + gs;
#pragma unroll
        for (int k = 0; k < NV; ++k) nv[k] = src[k * n];
    };
    fetch(0);
#pragma unroll 1
    for (int f0 = 0; f0 < a.frames; f0 += FC) {
        const int nf = min(FC, a.frames - f0);
        __syncthreads();
        if (tid < nf) {
            const float t = a.times ? a.times[f0 + tid] : a.t0;
            ft[tid] = t;
            if (spline) {
                float N[4];
                spans[tid] = spline_basis<float>(a.n_ctrl, fminf(fmaxf(t, 0.0f), 1.0f), N);
                for (int r = 0; r < 4; ++r) weights[tid][r] = N[r];
            }
            if (SH && !DYN) {
                const CamD c = load_camera(a.poses + 7 * (f0 + tid));
                for (int i = 0; i < 3; ++i)
                    centre[tid][i] = c.ok ? static_cast<float>(-(c.R[0 * 3 + i] * c.t[0] + c.R[1 * 3 + i] * c.t[1] +
                                                                 c.R[2 * 3 + i] * c.t[2]))
                                          : 0.0f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int fi = 0; fi < nf; ++fi) {
            const uint32_t cnt = ncnt;
            float x[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) x[k] = nv[k];
            if (f0 + fi + 1 < a.frames) fetch(f0 + fi + 1);
            if (ctrl_out) {
                const int sp = __builtin_amdgcn_readfirstlane(spans[fi]);
                if (sp != win) {
                    flush_window();
                    win = sp;
                }
            }
            if (!cnt) continue;
            const float t = ft[fi];
            const double t1 = t, t2 = t1 * t1, t3 = t2 * t1;
            float go[14];
            if (DYN) {
                for (int k = 0; k < 14; ++k) go[k] = x[k];
            } else {
                for (int k = 0; k < 9; ++k) go[k] = x[k];
                go[9] = 0.0f;
                for (int k = 9; k < 13; ++k) go[k + 1] = x[k];
            }
            for (int k = 0; k < 14; ++k) acc[k] += go[k];
            if constexpr (DYN) {
                if (ctrl_out)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int k = 0; k < 3; ++k) win_acc[3 * r + k] += weights[fi][r] * go[k];
                else if (a.mean_coeffs)
                    for (int k = 0; k < 3; ++k) {
                        win_acc[k] += go[k] * t1;
                        win_acc[3 + k] += go[k] * t2;
                        win_acc[6 + k] += go[k] * t3;
                    }
                if (a.scale_coeffs)
                    for (int k = 0; k < 3; ++k) {
                        sc[k] += go[3 + k] * t1;
                        sc[3 + k] += go[3 + k] * t2;
                        sc[6 + k] += go[3 + k] * t3;
                    }
                if (a.quat_coeffs)
                    for (int k = 0; k < 4; ++k) {
                        qc[k] += go[6 + k] * t1;
                        qc[4 + k] += go[6 + k] * t2;
                        qc[8 + k] += go[6 + k] * t3;
                    }
            } else if (a.mean_coeffs) {
                for (int k = 0; k < 3; ++k) {
                    cubic[k] += go[k] * t1;
                    cubic[3 + k] += go[k] * t2;
                    cubic[6 + k] += go[k] * t3;
                }
            }
            if constexpr (SH) {
                float d[3];
                if constexpr (DYN) {
                    for (int j = 0; j < 3; ++j) d[j] = x[14 + j];
                } else {
                    float v[3];
                    for (int k = 0; k < 3; ++k)
                        v[k] = mu0[k] + t * (mc[k] + t * (mc[3 + k] + t * mc[6 + k])) - centre[fi][k];
                    const float vn = sqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
                    const float iv = vn > 0.0f ? 1.0f / vn : 0.0f;
                    for (int j = 0; j < 3; ++j) d[j] = v[j] * iv;
                }
                float Y[15];
                sh_eval<float>(3, d[0], d[1], d[2], Y, nullptr);
                auto add = [&](auto from, auto to) {
#pragma unroll
                    for (int k = decltype(from)::value; k < decltype(to)::value; ++k)
#pragma unroll
                        for (int c = 0; c < 3; ++c) sh[3 * k + c] += Y[k] * go[11 + c];
                };
                add(std::integral_constant<int, 0>{}, std::integral_constant<int, 3>{});
                if (a.sh_degree >= 2) add(std::integral_constant<int, 3>{}, std::integral_constant<int, 8>{});
                if (a.sh_degree >= 3) add(std::integral_constant<int, 8>{}, std::integral_constant<int, 15>{});
            }
        }
    }
    if (!live) return;
    if (ctrl_out) flush_window();
    auto put = [&](float* dst, int64_t idx, double v) {
        if (!dst) return;
        if (a.accumulate) dst[idx] += static_cast<float>(v);
        else dst[idx] = static_cast<float>(v);
    };
    double gsq[7];
    if (DYN) {
        for (int k = 0; k < 7; ++k) gsq[k] = acc[3 + k];
    } else {
        static_shape_adjoint<T>(a, g, acc + 3, gsq);
    }
    for (int k = 0; k < 3; ++k) {
        if (a.n_ctrl == 0) put(a.g_means, k * n + g, acc[k]);
        put(a.g_log_scales, k * n + g, gsq[k]);
        put(a.g_colors, k * n + g, acc[11 + k]);
    }
    for (int k = 0; k < 4; ++k) put(a.g_quats, k * n + g, gsq[3 + k]);
    put(a.g_opacity, g, acc[10]);
    if constexpr (DYN) {
        if (a.mean_coeffs)
            for (int k = 0; k < 9; ++k) put(a.g_coeffs, k * n + g, win_acc[k]);
        if (a.scale_coeffs)
            for (int k = 0; k < 9; ++k) put(a.g_scale_coeffs, k * n + g, sc[k]);
        if (a.quat_coeffs)
            for (int k = 0; k < 12; ++k) put(a.g_quat_coeffs, k * n + g, qc[k]);
    } else if (a.mean_coeffs) {
        for (int k = 0; k < 9; ++k) put(a.g_coeffs, k * n + g, cubic[k]);
    }
    if constexpr (SH) {
#pragma unroll
        for (int k = 0; k < 45; ++k)
            if (k < 3 * sh_count(a.sh_degree)) put(a.g_sh, static_cast<int64_t>(k) * n + g, sh[k]);
    }
}

// The one-kernel form of the adjoint with dynamics or SH.  SPLIT waves share
// each Gaussian: wave h of a workgroup takes the h-th
// contiguous part of the frames for the workgroup's 64 Gaussians, and the
// parts' accumulators are added in a fixed order at the end.  Shorter parts
// keep more waves in flight for this latency-bound kernel and leave a shorter
// tail when the last workgroups run alone.  The dynamic variant keeps one
// wave per Gaussian (its control-point window adds to memory as it moves) and
// the SH variant two parts (its coefficient accumulators take LDS).
template <bool DYN, bool SH>
constexpr int pb_split() { return DYN ? 1 : 2; }
template <bool DYN, bool SH>
constexpr int pb_threads() { return DYN ? 128 : 64 * pb_split<DYN, SH>(); }

template <bool DYN, bool SH, typename T>
__global__ __launch_bounds__((pb_threads<DYN, SH>())) void k_project_bwd(Args a) {
    if (overflowed(a.status)) return;
    using LA = AccLayout<DYN>;
    constexpr int PB_THREADS = pb_threads<DYN, SH>();
    constexpr int SPLIT = pb_split<DYN, SH>();
    constexpr int GPB = PB_THREADS / SPLIT;  // Gaussians per workgroup
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int h = tid / GPB;                 // which part of the frames
    const int64_t g = static_cast<int64_t>(blockIdx.x) * GPB + (tid % GPB);
    const bool live = g < a.n;
    const int64_t n = a.n;
    const int fpart = (a.frames + SPLIT - 1) / SPLIT;
    const int fb = h * fpart < a.frames ? h * fpart : a.frames;
    const int fe = fb + fpart < a.frames ? fb + fpart : a.frames;
    __shared__ double red[PB_THREADS / 64][4];
    // per-thread gradient accumulators (FP64) live in LDS, see AccLayout
    __shared__ double acc[LA::N][PB_THREADS];
    // cameras of a chunk of frames (R 0-8, t 9-11, centre 12-14) and the
    // per-wave pose sums of each of its frames
    constexpr int FC = 32;
    __shared__ float cam[SPLIT][FC][15];
    __shared__ float wpose[SPLIT][FC][PB_THREADS / 64 / SPLIT][12];
    __shared__ double iacc[4][PB_THREADS];  // intrinsics gradient, summed over frames
    for (int k = 0; k < 4; ++k) iacc[k][tid] = 0.0;
    // SH coefficient gradients (FP32: at most a few hundred frames are summed; in
    // FP64, as the two-kernel form sums them, 188 -> 245 us for 20 frames of 100k
    // Gaussians with degree 3)
    __shared__ float acc_sh[SH ? 45 : 1][PB_THREADS];
    for (int k = 0; k < LA::N; ++k) acc[k][tid] = 0.0;
    if (SH)
        for (int k = 0; k < 3 * sh_count(a.sh_degree); ++k) acc_sh[k][tid] = 0.0f;
    // control-point window: gradients of points win .. win + 3, flushed to
    // memory (added) when a frame falls in another knot span
    int win = -1;
    const bool spline = DYN && a.n_ctrl > 0 && a.g_ctrl != nullptr;
    auto flush_window = [&]() {
        if (win < 0) return;
        for (int r = 0; r < 4; ++r)
            for (int k = 0; k < 3; ++k) {
                float* dst = a.g_ctrl + (static_cast<int64_t>(win + r) * 3 + k) * n + g;
                *dst += static_cast<float>(acc[LA::WIN + 3 * r + k][tid]);
                acc[LA::WIN + 3 * r + k][tid] = 0.0;
            }
    };
    if (spline && live && !a.accumulate)
        for (int64_t i = 0; i < static_cast<int64_t>(a.n_ctrl) * 3; ++i) a.g_ctrl[i * n + g] = 0.0f;

    // a static Gaussian's shape (scales, rotation, 3D covariance, opacity) is
    // the same in every frame
    AdjIn Pstatic = {};
    if (!DYN && live) static_inputs(a, g, Pstatic);
    // the next frame's count, slot offset and record are loaded one frame ahead
    uint32_t cnt_n = 0u, base_n = 0u;
    Record rec_n = {};
    // (unconditional loads: no wait on the count before the record is requested)
    auto fetch = [&](int f) {
        const int64_t i = static_cast<int64_t>(f) * a.n + (live ? g : 0);
        cnt_n = live ? a.gcnt[i] : 0u;
        base_n = live ? a.goff[i] : 0u;
        rec_n = a.rec[i];
    };
    if (fb < fe) fetch(fb);
#pragma unroll 1
    for (int c0 = 0; c0 < fpart; c0 += FC) {  // the same chunk count in every wave (uniform barriers)
        const int f0 = fb + c0;
        const int nf = fe - f0 < FC ? (fe - f0 > 0 ? fe - f0 : 0) : FC;
        __syncthreads();  // the previous chunk's cameras and pose sums are consumed
        for (int q = tid; q < SPLIT * FC; q += PB_THREADS) {
            const int hh = q / FC, fi = q % FC;
            const int ff = hh * fpart + c0 + fi;
            const int fend = (hh + 1) * fpart < a.frames ? (hh + 1) * fpart : a.frames;
            if (ff < fend) {
                const CamD c = load_camera(a.poses + 7 * ff);
                for (int k = 0; k < 9; ++k) cam[hh][fi][k] = c.ok ? static_cast<float>(c.R[k]) : 0.0f;
                for (int k = 0; k < 3; ++k) cam[hh][fi][9 + k] = c.ok ? static_cast<float>(c.t[k]) : 0.0f;
                for (int i = 0; i < 3; ++i)
                    cam[hh][fi][12 + i] = c.ok ? static_cast<float>(-(c.R[0 * 3 + i] * c.t[0] +
                                                                      c.R[1 * 3 + i] * c.t[1] + c.R[2 * 3 + i] * c.t[2]))
                                               : 0.0f;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int fi = 0; fi < nf; ++fi) {
            const int f = f0 + fi;
            uint32_t cnt = cnt_n;
            const uint32_t base = base_n;
            const Record rec = rec_n;
            if (f + 1 < fe) fetch(f + 1);
            if (static_cast<int64_t>(base) + cnt > a.k_cap) cnt = 0u;  // only after an internal error
            const float* camR = cam[h][fi];
            const float* camT = cam[h][fi] + 9;
            const float* camC = cam[h][fi] + 12;
            float pose[12];
            for (int k = 0; k < 12; ++k) pose[k] = 0.0f;
            if (cnt) {
                // PU records per round, loads issued together (past the end
                // they repeat a valid record and are not added), summed in
                // order k = 0, 1, ...; the first round is requested before the
                // frame's projection inputs are computed, which do not need it.
                // Only the records the adjoint wrote this pass (bit set in
                // pused) are added: the others belong to entries behind their
                // tile's last contributor and hold stale values.
                constexpr uint32_t PU = 8;
                float r[PU][PART];
                uint32_t w0 = 0u, w1 = 0u;  // pused words holding the round's bits
                auto load_round = [&](uint32_t k0) {
                    const uint32_t wi = (base + k0) >> 5;
                    w0 = a.pused[wi];
                    w1 = a.pused[wi + 1];
#pragma unroll
                    for (uint32_t u = 0; u < PU; ++u) {
                        const uint32_t k = k0 + u < cnt ? k0 + u : k0;
                        const float* pp = a.part + static_cast<int64_t>(base + k) * PART;
#pragma unroll
                        for (int m = 0; m < PART; ++m) r[u][m] = pp[m];
                    }
                };
                load_round(0);
                const float t = a.times ? a.times[f] : a.t0;
                AdjIn P = Pstatic;
                if (DYN) shape_inputs<T>(a, g, t, P);
                frame_inputs<DYN, T>(a, g, rec, camR, camT, t, P);
                double dd[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
                for (uint32_t k0 = 0;;) {
                    const uint32_t bits = static_cast<uint32_t>(
                        ((static_cast<uint64_t>(w1) << 32) | w0) >> ((base + k0) & 31u));
#pragma unroll
                    for (uint32_t u = 0; u < PU; ++u)
                        if (k0 + u < cnt && ((bits >> u) & 1u))
#pragma unroll
                            for (int m = 0; m < PART; ++m) dd[m] += r[u][m];
                    k0 += PU;
                    if (k0 >= cnt) break;
                    load_round(k0);
                }
                float d[9];
                for (int k = 0; k < 9; ++k) d[k] = static_cast<float>(dd[k]);
                float go[14], gi[4];
                projection_adjoint<!DYN>(a, camR, P, d, go, pose, gi);
                if (a.g_intr)
                    for (int k = 0; k < 4; ++k) iacc[k][tid] += gi[k];
                if (SH) {
                    float dv[3];
                    const float dc[3] = {go[11], go[12], go[13]};
                    sh_adjoint<PB_THREADS, T>(a, g, P, camC, dc, acc_sh, tid, dv);
                    for (int j = 0; j < 3; ++j) {
                        go[j] += dv[j];
                        // C = -Rc^T tc, dL/dC = -dv: dL/dtc = Rc dv, dL/dRc[j][i] = tc[j] dv[i]
                        pose[9 + j] += camR[j * 3 + 0] * dv[0] + camR[j * 3 + 1] * dv[1] + camR[j * 3 + 2] * dv[2];
                        for (int i = 0; i < 3; ++i) pose[j * 3 + i] += camT[j] * dv[i];
                    }
                }
                for (int k = 0; k < 14; ++k) acc[k][tid] += go[k];
                const double t1 = t, t2 = t1 * t1, t3 = t2 * t1;
                if (a.mean_coeffs)
                    for (int k = 0; k < 3; ++k) {
                        acc[LA::CUBIC + k][tid] += go[k] * t1;
                        acc[LA::CUBIC + 3 + k][tid] += go[k] * t2;
                        acc[LA::CUBIC + 6 + k][tid] += go[k] * t3;
                    }
                if (DYN) {
                    if (spline) {
                        if (P.span != win) {
                            flush_window();
                            win = P.span;
                        }
                        for (int r = 0; r < 4; ++r)
                            for (int k = 0; k < 3; ++k) acc[LA::WIN + 3 * r + k][tid] += P.N[r] * go[k];
                    }
                    if (a.scale_coeffs)
                        for (int k = 0; k < 3; ++k) {
                            acc[LA::SCALE + k][tid] += go[3 + k] * t1;
                            acc[LA::SCALE + 3 + k][tid] += go[3 + k] * t2;
                            acc[LA::SCALE + 6 + k][tid] += go[3 + k] * t3;
                        }
                    if (a.quat_coeffs)
                        for (int k = 0; k < 4; ++k) {
                            acc[LA::QUAT + k][tid] += go[6 + k] * t1;
                            acc[LA::QUAT + 4 + k][tid] += go[6 + k] * t2;
                            acc[LA::QUAT + 8 + k][tid] += go[6 + k] * t3;
                        }
                }
            }
            if (a.g_poses) {  // wave sums of this frame's pose contributions
                float v[16];
#pragma unroll
                for (int k = 0; k < 12; ++k) v[k] = pose[k];
#pragma unroll
                for (int k = 12; k < 16; ++k) v[k] = 0.0f;
                const float x = reduce_scatter16(v, lane);
                const int idx = reduce_scatter16_index(lane);
                if ((lane & 3) == 0 && idx < 12) wpose[h][fi][w % (PB_THREADS / 64 / SPLIT)][idx] = x;
            }
        }
        if (a.g_poses) {
            __syncthreads();
            constexpr int WPH = PB_THREADS / 64 / SPLIT;  // waves per part
            for (int q = tid; q < SPLIT * FC * 12; q += PB_THREADS) {
                const int hh = q / (FC * 12), r = q % (FC * 12), fi = r / 12, k = r % 12;
                const int ff = hh * fpart + c0 + fi;
                const int fend = (hh + 1) * fpart < a.frames ? (hh + 1) * fpart : a.frames;
                if (ff >= fend) continue;
                double v = 0.0;
                for (int ww = 0; ww < WPH; ++ww) v += static_cast<double>(wpose[hh][fi][ww][k]);
                a.pose_part[(static_cast<int64_t>(blockIdx.x) * a.frames + ff) * 12 + k] = v;
            }
        }
    }
    if (a.g_intr) {  // uniform: every thread takes part in the block reduction
        __syncthreads();
        for (int k = 0; k < 4; ++k) {
            const double v = wave_sum_f64(iacc[k][tid]);
            if (lane == 0) red[w][k] = v;
        }
        __syncthreads();
        if (tid < 4) {
            double v = 0.0;
            for (int ww = 0; ww < PB_THREADS / 64; ++ww) v += red[ww][tid];
            a.intr_part[static_cast<int64_t>(blockIdx.x) * 4 + tid] = v;
        }
    }
    if (SPLIT > 1) {  // add the later parts' accumulators to part 0's, in order
        __syncthreads();
        if (h == 0) {
            for (int k = 0; k < LA::N; ++k) {
                double v = acc[k][tid];
                for (int hh = 1; hh < SPLIT; ++hh) v += acc[k][tid + hh * GPB];
                acc[k][tid] = v;
            }
            if (SH)
                for (int k = 0; k < 3 * sh_count(a.sh_degree); ++k) {
                    float v = acc_sh[k][tid];
                    for (int hh = 1; hh < SPLIT; ++hh) v += acc_sh[k][tid + hh * GPB];
                    acc_sh[k][tid] = v;
                }
        }
    }
    if (!live || h != 0) return;
    if (spline) flush_window();
    auto put = [&](float* dst, int64_t idx, double v) {
        if (!dst) return;
        if (a.accumulate) dst[idx] += static_cast<float>(v);
        else dst[idx] = static_cast<float>(v);
    };
    double gsq[7];  // log-scales, quaternion
    if (DYN) {
        for (int k = 0; k < 7; ++k) gsq[k] = acc[3 + k][tid];
    } else {  // dL/dSig summed over the frames, through the shape once
        double Gs[6];
        for (int k = 0; k < 6; ++k) Gs[k] = acc[3 + k][tid];
        static_shape_adjoint<T>(a, g, Gs, gsq);
    }
    for (int k = 0; k < 3; ++k) {
        if (a.n_ctrl == 0) put(a.g_means, k * n + g, acc[k][tid]);
        put(a.g_log_scales, k * n + g, gsq[k]);
        put(a.g_colors, k * n + g, acc[11 + k][tid]);
    }
    for (int k = 0; k < 4; ++k) put(a.g_quats, k * n + g, gsq[3 + k]);
    put(a.g_opacity, g, acc[10][tid]);
    if (a.mean_coeffs)
        for (int c = 0; c < 3; ++c)
            for (int k = 0; k < 3; ++k) put(a.g_coeffs, (c * 3 + k) * n + g, acc[LA::CUBIC + c * 3 + k][tid]);
    if (DYN && a.scale_coeffs)
        for (int c = 0; c < 3; ++c)
            for (int k = 0; k < 3; ++k) put(a.g_scale_coeffs, (c * 3 + k) * n + g, acc[LA::SCALE + c * 3 + k][tid]);
    if (DYN && a.quat_coeffs)
        for (int c = 0; c < 3; ++c)
            for (int k = 0; k < 4; ++k) put(a.g_quat_coeffs, (c * 4 + k) * n + g, acc[LA::QUAT + c * 4 + k][tid]);
    if (SH)
        for (int k = 0; k < 3 * sh_count(a.sh_degree); ++k) put(a.g_sh, static_cast<int64_t>(k) * n + g, acc_sh[k][tid]);
}

// Sums of V values over the projection adjoint's workgroups, part[b * stride + k]
// for k < V, in a fixed order: groups of V threads (whose loads are contiguous)
// take every GROUPS-th workgroup, then the groups are added in order.  The sums
// are in out[0, V) for every thread afterwards.
constexpr int FIN_THREADS = 1024;

template <int V>
__device__ __forceinline__ void sum_parts(const double* part, int64_t stride, int64_t n_blocks, double* red,
                                          double* out) {
    constexpr int GROUPS = FIN_THREADS / V;
    const int q = threadIdx.x / V, k = threadIdx.x % V;
    if (q < GROUPS) {
        double v = 0.0;
#pragma unroll 4
        for (int64_t b = q; b < n_blocks; b += GROUPS) v += part[b * stride + k];
        red[q * V + k] = v;
    }
    __syncthreads();
    const int used = n_blocks < GROUPS ? static_cast<int>(n_blocks) : GROUPS;
    if (threadIdx.x < V) {
        double v = 0.0;
        for (int g = 0; g < used; ++g) v += red[g * V + threadIdx.x];
        out[threadIdx.x] = v;
    }
    __syncthreads();
}

// Workgroup f < pose_frames: the frame's pose gradient, its sums of dL/dRc and
// dL/dtc mapped to the unnormalised pose quaternion and translation.  The
// workgroups after them: the intrinsics gradient (one), or, with per-frame
// partials frame_intr [frame][n_blocks][4], each frame's sum, left in the
// frame's first partial (one per frame; k_intr_frames adds them).
__global__ __launch_bounds__(FIN_THREADS) void k_adjoint_finalize(Args a, int64_t n_blocks, int pose_frames,
                                                                  double* frame_intr) {
    __shared__ double red[FIN_THREADS], acc[12];
    const int f = blockIdx.x;
    if (f < pose_frames) {
        sum_parts<12>(a.pose_part + static_cast<int64_t>(f) * 12, static_cast<int64_t>(a.frames) * 12, n_blocks, red,
                      acc);
        if (threadIdx.x != 0) return;
        double G[9];
        for (int k = 0; k < 9; ++k) G[k] = acc[k];
        const CamD cam = load_camera(a.poses + 7 * f);
        double dq[4] = {0, 0, 0, 0};
        if (cam.ok) quat_grad(cam.qh, cam.qn, G, dq);
        float* out = a.g_poses + 7 * f;
        const bool bad = overflowed(a.status);
        for (int k = 0; k < 4; ++k) out[k] = bad ? 0.0f : static_cast<float>(dq[k]);
        for (int k = 0; k < 3; ++k) out[4 + k] = bad ? 0.0f : static_cast<float>(acc[9 + k]);
    } else if (frame_intr) {
        double* part = frame_intr + static_cast<int64_t>(f - pose_frames) * n_blocks * 4;
        sum_parts<4>(part, 4, n_blocks, red, acc);
        if (threadIdx.x < 4) part[threadIdx.x] = acc[threadIdx.x];
    } else {
        sum_parts<4>(a.intr_part, 4, n_blocks, red, acc);
        if (threadIdx.x >= 4) return;
        const float g = overflowed(a.status) ? 0.0f : static_cast<float>(acc[threadIdx.x]);
        if (a.accumulate) a.g_intr[threadIdx.x] += g;
        else a.g_intr[threadIdx.x] = g;
    }
}

__global__ __launch_bounds__(FIN_THREADS) void k_intr_frames(Args a, int64_t n_blocks, const double* frame_intr) {
    __shared__ double red[FIN_THREADS], acc[12];
    sum_parts<4>(frame_intr, n_blocks * 4, a.frames, red, acc);
    if (threadIdx.x >= 4) return;
    const float g = overflowed(a.status) ? 0.0f : static_cast<float>(acc[threadIdx.x]);
    if (a.accumulate) a.g_intr[threadIdx.x] += g;
    else a.g_intr[threadIdx.x] = g;
}

// Do the Gaussians meet many tiles each?  The host knows the workspace's
// capacity, which callers size to their scene; where it is generous the forms
// for large Gaussians give the same results up to the order of sums, more slowly.
// Above the line the static adjoint of few frames takes LARGE, and of four and
// more the two-kernel form, whose lanes are (frame, Gaussian) pairs, which fill
// the chip with fewer Gaussians: 50 960x540 frames of 20k Gaussians of 33 tiles
// 1,094 us in one kernel, 580 in two, of 50k of 15 tiles 860 and 644, 500 640x360
// frames of 100 of 41 tiles 6,159 and 341, 12 960x540 frames of 80k of 16 tiles 319
// and 274; 16 1080p frames of 500k of ten tiles 1,068 and 1,202, 50 960x540 frames
// of 200k of ten tiles 1,534 and 1,563, of four 620 and 808.  Fewer Gaussians gain
// from fewer tiles on: 50 frames of 2,000 of seven 184 and 62 us, 100 320x240 frames
// of 300 of seven 170 and 72; four 128x128 frames of 500 of three 14 and 19.
static bool large_gaussians(const Args& a) {
    const int64_t line = a.n <= 16384 ? 8 : a.n <= 65536 ? 16 : 32;  // of capacity, per (frame, Gaussian)
    return a.k_cap / (line * a.frames) >= a.n;
}

// Gaussians per workgroup of each variant.
template <bool DYN, bool SH>
constexpr int pb_gaussians() { return pb_threads<DYN, SH>() / pb_split<DYN, SH>(); }
constexpr int STATIC_GAUSSIANS = 64;  // of k_adjoint_static
static_assert(pb_gaussians<false, true>() >= STATIC_GAUSSIANS && pb_gaussians<true, false>() >= STATIC_GAUSSIANS &&
                  pb_gaussians<true, true>() >= STATIC_GAUSSIANS,
              "the static kernel has the most workgroups");

// Upper bound over the variants.
int64_t project_bwd_blocks(int64_t n) {
    return (n + STATIC_GAUSSIANS - 1) / STATIC_GAUSSIANS;
}

static int64_t blocks_for(int64_t n, bool dyn, bool sh) {
    const int gpb = dyn ? (sh ? pb_gaussians<true, true>() : pb_gaussians<true, false>())
                        : (sh ? pb_gaussians<false, true>() : STATIC_GAUSSIANS);
    return (n + gpb - 1) / gpb;
}

template <int SPLIT, bool LARGE, typename T>
static void launch_static_split(const Args& a, dim3 grid, hipStream_t stream) {
    const dim3 block(64 * SPLIT);
    if (a.mean_coeffs) hipLaunchKernelGGL((k_adjoint_static<SPLIT, true, T, LARGE>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_adjoint_static<SPLIT, false, T, LARGE>), grid, block, 0, stream, a);
}

template <typename T>
static void launch_static(const Args& a, dim3 grid, hipStream_t stream) {
    // four parts of the frames per 64 Gaussians where there are four frames
    if (a.frames >= 4) launch_static_split<4, false, T>(a, grid, stream);
    else if (!large_gaussians(a)) launch_static_split<1, false, T>(a, grid, stream);
    else if (a.frames == 3) launch_static_split<3, true, T>(a, grid, stream);
    else if (a.frames == 2) launch_static_split<2, true, T>(a, grid, stream);
    else launch_static_split<1, true, T>(a, grid, stream);
}

// The two-kernel form of the adjoint with dynamics or SH, if the store fits in
// the sort's key buffers and the intrinsics partials behind the pose partials;
// false if not.  The projection's workspace holds 12 doubles per frame and 64
// Gaussians for the pose partials, of which this form's 256 take a quarter.
template <bool DYN, bool SH, typename T>
static bool launch_two_kernels(const Args& a, FrameStore& store, hipStream_t stream) {
    constexpr int64_t NV = frame_values<DYN, SH>();
    const int64_t blocks = (a.n + 255) / 256;
    store.stride = (NV * a.n + 63) / 64 * 64;
    const int64_t fit = static_cast<int64_t>(sizeof(KeySlot)) * a.k_cap / 4 / store.stride;
    if (2 * fit < a.frames || blocks * 16 > project_bwd_blocks(a.n) * 12) return false;
    store.lo = reinterpret_cast<float*>(a.kv);
    store.hi = reinterpret_cast<float*>(a.tkv);
    store.lo_frames = static_cast<int>(fit < a.frames ? fit : a.frames);
    store.blocks = static_cast<int>(blocks);
    store.intr = a.pose_part + blocks * a.frames * 12;
    const dim3 grid(XCDS * xcd_share(store.blocks, a.frames));
    hipLaunchKernelGGL((k_adjoint_frames<DYN, SH, T>), grid, dim3(256), 0, stream, a, store);
    hipLaunchKernelGGL((k_adjoint_sum<DYN, SH, T>), dim3(static_cast<uint32_t>((a.n + 127) / 128)), dim3(128), 0, stream,
                       a, store);
    return true;
}

template <bool DYN, bool SH, typename T>
static void launch_adjoint(const Args& a, int64_t& nb, double*& frame_intr, hipStream_t stream) {
    FrameStore store;
    if (launch_two_kernels<DYN, SH, T>(a, store, stream)) {
        nb = store.blocks;
        frame_intr = store.intr;
        return;
    }
    nb = blocks_for(a.n, DYN, SH);
    hipLaunchKernelGGL((k_project_bwd<DYN, SH, T>), dim3(static_cast<uint32_t>(nb)), dim3(pb_threads<DYN, SH>()), 0,
                       stream, a);
}

template <typename T>
static void launch_adjoint_as(const Args& a, int64_t& nb, double*& frame_intr, hipStream_t stream) {
    const bool dyn = a.n_ctrl > 0 || a.scale_coeffs || a.quat_coeffs, sh = a.sh_degree > 0;
    if (dyn && sh) launch_adjoint<true, true, T>(a, nb, frame_intr, stream);
    else if (dyn) launch_adjoint<true, false, T>(a, nb, frame_intr, stream);
    else if (sh) launch_adjoint<false, true, T>(a, nb, frame_intr, stream);
    else if (FrameStore store; a.frames >= 4 && large_gaussians(a) && launch_two_kernels<false, false, T>(a, store, stream)) {
        nb = store.blocks;
        frame_intr = store.intr;
    } else {
        nb = blocks_for(a.n, false, false);
        launch_static<T>(a, dim3(static_cast<uint32_t>(nb)), stream);
    }
}

hipError_t launch_project_bwd(const Args& a, hipStream_t stream) {
    int64_t nb = 0;
    double* frame_intr = nullptr;
    if (a.n > 0) {
        if (a.dtype == GV_BF16) launch_adjoint_as<uint16_t>(a, nb, frame_intr, stream);
        else launch_adjoint_as<float>(a, nb, frame_intr, stream);
    }
    const int pose_frames = a.g_poses ? a.frames : 0, intr = !a.g_intr ? 0 : frame_intr ? a.frames : 1;
    if (pose_frames + intr > 0)
        hipLaunchKernelGGL(k_adjoint_finalize, dim3(static_cast<uint32_t>(pose_frames + intr)), dim3(FIN_THREADS), 0,
                           stream, a, nb, pose_frames, a.g_intr ? frame_intr : nullptr);
    if (a.g_intr && frame_intr) hipLaunchKernelGGL(k_intr_frames, dim3(1), dim3(FIN_THREADS), 0, stream, a, nb, frame_intr);
    return hipGetLastError();
}

}  // namespace gv
