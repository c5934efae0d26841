// Camera-motion Neural ODE (Eq. 1, Sec. 3.4): fused MLP + RK4 forward and its
// discrete adjoint, each in one workgroup of four waves.
//
// The integration is a serial chain of (F-1) * S * 4 evaluations of the
// 8 -> 64 -> 64 -> 7 tanh MLP, so latency, not throughput, is what matters: the
// instructions on the chain, the exchanges between lanes and nothing else.
//  - The hidden-to-hidden product is the longest link.  Every wave computes the
//    whole first hidden layer itself, lane u unit u, so each 16-lane row holds
//    16 of its values; lane (row c, l) of wave w then sums the terms of row c
//    for unit 16 w + l, reading them as row broadcasts of the DPP operand (no
//    LDS, no barrier), and two row swaps add the four rows.  So the product's
//    4,096 terms are 16 instructions on each of a CU's four SIMDs.
//  - The 7 outputs: row c of a wave sums its wave's 16 units for outputs 2 c
//    and 2 c + 1; the four waves' sums meet in LDS, the one exchange (one
//    barrier) of an evaluation.
//  - The state needs no exchange: the 8 lanes of output i hold component i of
//    the state in every wave, and the RK4 arithmetic is done for one component
//    per lane.  The next input goes to all lanes as scalars (readlane).
//  - Nothing else is on the chain: poses are written from the recorded states
//    afterwards, the adjoint's pose cotangents are formed before it starts, and
//    the next evaluation's recorded activations are requested one ahead.
// The state z is carried in FP64, the MLP runs in FP32.  The forward pass
// records every evaluation's input and both hidden activations so that the
// adjoint needs no recomputation; the adjoint's chain records each
// evaluation's cotangents, and the parameter gradient (outer products summed
// over the evaluations) is formed from those records by parallel kernels.
// 100 frames, 4 substeps (1,584 evaluations): forward 885 us in one wave, 478 us
// so; adjoint 701 -> 477 us.
#include "gv_internal.h"

namespace gv {

constexpr int ODE_H = 64;
constexpr int ODE_S = 7;
constexpr int ODE_REC = 8 + ODE_H + ODE_H;  // x, h1, h2 of one evaluation
static_assert(ODE_REC % 4 == 0, "records start on 16-byte boundaries");
// offsets of the parameter blocks in theta
constexpr int OFF_W1 = 0, OFF_B1 = 512, OFF_W2 = 576, OFF_B2 = 4672, OFF_W3 = 4736, OFF_B3 = 5184, N_THETA = 5191;

constexpr int ODE_ADJ = ODE_H + ODE_H + 8;  // da1, da2, dy (+ pad) of one evaluation
constexpr int ODE_CHUNKS = 64;              // partial sums of the parameter gradient

struct OdeLayout {
    size_t evals, chunks, chunk;
    size_t acts, zf, adj, part, total;
};

static inline size_t ode_align(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

OdeLayout ode_layout(int frames, int substeps) {
    OdeLayout L;
    L.evals = static_cast<size_t>(frames - 1) * substeps * 4;
    L.chunks = L.evals < ODE_CHUNKS ? (L.evals > 0 ? L.evals : 1) : ODE_CHUNKS;
    L.chunk = (L.evals + L.chunks - 1) / L.chunks;
    L.acts = 0;
    L.zf = ode_align(L.evals * ODE_REC * sizeof(float));
    L.adj = L.zf + ode_align(static_cast<size_t>(frames) * ODE_S * sizeof(double));
    L.part = L.adj + ode_align(L.evals * ODE_ADJ * sizeof(float));
    L.total = L.part + ode_align(L.chunks * N_THETA * sizeof(float));
    return L;
}

constexpr int ODE_WG = 256;

// tanh: for small |x| an odd polynomial (a weighted least-squares fit of
// (tanh x / x - 1) / x^2 on [0, 0.55]; with its coefficients rounded to FP32 within
// 4.4e-9 of tanh x; as evaluated within 0.6 ulp of the result, measured), else
// 1 - 2 / (1 + e^2|x|) by the hardware's exp2 and reciprocal (1.6 ulp measured, just
// above 0.55; 2.7 if both were off by one).  Both are computed and one selected: a
// third of the instructions of the library's branching form, which was a quarter
// of an evaluation.
__device__ __forceinline__ float ode_tanh(float x) {
    const float a = fabsf(x), u = x * x;
    float q = -6.274235900e-03f;
    q = __builtin_fmaf(q, u, 2.107167616e-02f);
    q = __builtin_fmaf(q, u, -5.385230854e-02f);
    q = __builtin_fmaf(q, u, 1.333258599e-01f);
    q = __builtin_fmaf(q, u, -3.333331645e-01f);
    float small = __builtin_fmaf(x * u, q, x);
    const float e = __builtin_amdgcn_exp2f(a * 2.8853900817779268f);  // e^(2a)
    float large = __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
    asm volatile("" : "+v"(small), "+v"(large));  // both, and a select: a branch costs more than either
    return a < 0.55f ? small : copysignf(large, x);
}

// acc + sum over k of w[k] times lane k of the 16-lane row, in order: 16 FMAs
// whose first operand is a row broadcast.  Written out because the compiler
// keeps the broadcast a move of its own, with a wait between the two: 48 issue
// slots instead of 16.  (The leading wait covers a value written just before.)
__device__ __forceinline__ float row_dot(const float (&w)[16], float x, float acc) {
    asm("s_nop 1\n"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
        "s_nop 1"
        : "+v"(acc)
        : "v"(x), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]), "v"(w[8]),
          "v"(w[9]), "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15]));
    return acc;
}

// Sum over the wave's four rows, in every one of them (each addition pairs the
// same two values in both: equal bits).
__device__ __forceinline__ float rows_sum(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums over the 16 lanes of each row of two values: lanes 0-7 get the first's,
// lanes 8-15 the second's.
__device__ __forceinline__ float row_sum2(float v0, float v1, int lane) {
    const bool b3 = lane & 8;
    const float keep = b3 ? v1 : v0, send = b3 ? v0 : v1;
    float x = keep + dpp_f(send, 0x128);
    x += dpp_f(x, 0x141);
    x += dpp_f(x, 0x4E);
    return x + dpp_f(x, 0xB1);
}

// Who does what: lane (= the unit whose first-layer value it forms), row c, the
// unit whose second-layer terms of row c it sums, output (or state component) i.
struct OdeLane {
    uint32_t w, lane, c, unit, i;
    __device__ OdeLane() {
        lane = threadIdx.x & 63;
        w = threadIdx.x >> 6;
        c = lane >> 4;
        unit = 16 * w + (lane & 15);
        i = lane >> 3;
    }
};

// The four waves' sums of component i, exchanged through one of two buffers in
// turn (a wave writes a buffer again only after a barrier that every wave
// reached with its reads of it done).
struct OdeExchange {
    float4 part[2][8];
    __device__ __forceinline__ float sum(int& turn, const OdeLane& L, float x) {
        reinterpret_cast<float*>(&part[turn][L.i])[L.w] = x;  // the component's lanes hold the same value
        __syncthreads();
        const float4 v = part[turn][L.i];
        turn ^= 1;
        return (v.x + v.y) + (v.z + v.w);
    }
};

// The N components of a value held by lanes 0, 8, 16, ..., as scalars.  All are
// read before the first use: read one at a time, each waits out the hazard
// between the lane read and its use.
template <int N>
__device__ __forceinline__ void components(float v, float (&s)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) s[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 8 * k));
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void write_pose(const double* z, float* pose) {
    const double n = sqrt(z[0] * z[0] + z[1] * z[1] + z[2] * z[2] + z[3] * z[3]);
    for (int k = 0; k < 4; ++k) pose[k] = static_cast<float>(z[k] / n);
    for (int k = 4; k < ODE_S; ++k) pose[k] = static_cast<float>(z[k]);
}

__global__ __launch_bounds__(ODE_WG) void k_ode_fwd(const float* __restrict__ theta, const float* __restrict__ z0,
                                                    int frames, int substeps, float* __restrict__ poses,
                                                    float* __restrict__ acts, double* zf) {
    const OdeLane L;
    __shared__ OdeExchange X;
    float w1[8], w2[16];
    for (int k = 0; k < 8; ++k) w1[k] = theta[OFF_W1 + L.lane * 8 + k];
    const float b1 = theta[OFF_B1 + L.lane];
    for (int k = 0; k < 16; ++k) w2[k] = theta[OFF_W2 + L.unit * ODE_H + 16 * L.c + k];
    const float b2 = L.c == 0 ? theta[OFF_B2 + L.unit] : 0.0f;
    const float w3a = theta[OFF_W3 + 2 * L.c * ODE_H + L.unit];
    const float w3b = 2 * L.c + 1 < ODE_S ? theta[OFF_W3 + (2 * L.c + 1) * ODE_H + L.unit] : 0.0f;
    const float b3 = L.i < ODE_S ? theta[OFF_B3 + L.i] : 0.0f;
    // component 7 of the input is the time: its "state" is set at every step
    // and its slope is 1
    const bool time = L.i == ODE_S;
    double z = L.i < ODE_S ? z0[L.i] : 0.0;
    const bool writer = L.w == 0 && (L.lane & 7) == 0 && !time;  // one lane per component
    if (writer) zf[L.i] = z;
    const double h = frames > 1 ? 1.0 / (static_cast<double>(substeps) * (frames - 1)) : 0.0;
    float* rec = acts;
    int turn = 0;
    auto eval = [&](double y) {
        const float x = static_cast<float>(y);
        float xs[8];
        components(x, xs);
        float a1 = b1;
#pragma unroll
        for (int k = 0; k < 8; ++k) a1 = __builtin_fmaf(w1[k], xs[k], a1);
        const float h1 = ode_tanh(a1);
        const float h2 = ode_tanh(rows_sum(row_dot(w2, h1, b2)));
        const float o = X.sum(turn, L, row_sum2(w3a * h2, w3b * h2, L.lane)) + b3;
        // the record, without branches: lanes that hold the same value write it
        // to the same place
        rec[static_cast<uint32_t>(L.i)] = x;
        rec[8u + L.lane] = h1;
        rec[8u + ODE_H + L.unit] = h2;
        rec += ODE_REC;
        return time ? 1.0f : o;
    };
    for (int f = 1; f < frames; ++f) {
        for (int s = 0; s < substeps; ++s) {
            if (time) z = (static_cast<double>(f - 1) * substeps + s) * h;
            const float k1 = eval(z);
            const float k2 = eval(z + 0.5 * h * k1);
            const float k3 = eval(z + 0.5 * h * k2);
            const float k4 = eval(z + h * k3);
            z = z + (h / 6.0) * (static_cast<double>(k1) + 2.0 * k2 + 2.0 * k3 + k4);
        }
        if (writer) zf[ODE_S * f + L.i] = z;
    }
    __threadfence();
    __syncthreads();
    for (int f = threadIdx.x; f < frames; f += ODE_WG) {
        double zk[ODE_S];
        for (int k = 0; k < ODE_S; ++k) zk[k] = __builtin_nontemporal_load(zf + ODE_S * f + k);
        write_pose(zk, poses + ODE_S * f);
    }
}

// Cotangent of the state from the cotangent of the pose (q/|q|, t).
__device__ __forceinline__ void pose_cotangent(const double* z, const float* dp, double out[ODE_S]) {
    const double n = sqrt(z[0] * z[0] + z[1] * z[1] + z[2] * z[2] + z[3] * z[3]);
    double qh[4], dot = 0.0;
    for (int k = 0; k < 4; ++k) {
        qh[k] = z[k] / n;
        dot += qh[k] * static_cast<double>(dp[k]);
    }
    for (int k = 0; k < 4; ++k) out[k] = (static_cast<double>(dp[k]) - qh[k] * dot) / n;
    for (int k = 4; k < ODE_S; ++k) out[k] = dp[k];
}

// The adjoint's chain.  Frame f's pose cotangent (f >= 1) waits in the first
// cotangent record of the frame's own evaluations, which are differentiated,
// and the record written, only after it has been taken; frame 0's in LDS.
__global__ __launch_bounds__(ODE_WG) void k_ode_bwd(const float* __restrict__ theta, int frames, int substeps,
                                                    const float* __restrict__ dposes, const float* __restrict__ acts,
                                                    const double* __restrict__ zf, float* adj,
                                                    float* __restrict__ dz0) {
    const OdeLane L;
    __shared__ OdeExchange X;
    __shared__ double cot0[8];
    float w2c[16], w3[ODE_S];
    for (int k = 0; k < ODE_S; ++k) w3[k] = theta[OFF_W3 + k * ODE_H + L.lane];
    for (int k = 0; k < 16; ++k) w2c[k] = theta[OFF_W2 + (16 * L.c + k) * ODE_H + L.unit];
    const float w1a = theta[OFF_W1 + L.unit * 8 + 2 * L.c];
    const float w1b = 2 * L.c + 1 < ODE_S ? theta[OFF_W1 + L.unit * 8 + 2 * L.c + 1] : 0.0f;
    auto cotangent = [&](int f) {
        return reinterpret_cast<double*>(adj + static_cast<size_t>(f - 1) * substeps * 4 * ODE_ADJ);
    };
    for (int f = threadIdx.x; f < frames; f += ODE_WG) {
        double c[ODE_S];
        pose_cotangent(zf + ODE_S * f, dposes + ODE_S * f, c);
        double* to = f > 0 ? cotangent(f) : cot0;
        for (int k = 0; k < ODE_S; ++k) to[k] = c[k];
    }
    __threadfence();
    __syncthreads();
    const bool comp = L.i < ODE_S;
    auto take = [&](int f) {  // component i of frame f's pose cotangent
        if (!comp) return 0.0;
        return f > 0 ? __builtin_nontemporal_load(cotangent(f) + L.i) : cot0[L.i];
    };
    double lam = take(frames - 1);
    if (frames > 1) {
        const double h = 1.0 / (static_cast<double>(substeps) * (frames - 1));
        // The evaluations are taken in descending order; this lane's hidden
        // activations of the next one are requested while the current one is
        // differentiated.
        int64_t e = static_cast<int64_t>(frames - 1) * substeps * 4 - 1;
        float nh1 = acts[e * ODE_REC + 8 + L.unit], nh2 = acts[e * ODE_REC + 8 + ODE_H + L.lane];
        int turn = 0;
        __syncthreads();  // every lane has its first cotangent
        auto vjp = [&](double dy) {
            const float h1 = nh1, h2 = nh2;
            const int64_t before = e > 0 ? e - 1 : 0;
            nh1 = acts[before * ODE_REC + 8 + L.unit];
            nh2 = acts[before * ODE_REC + 8 + ODE_H + L.lane];
            float* out = adj + e * ODE_ADJ;
            --e;
            const float dyf = static_cast<float>(dy);
            float dys[ODE_S];
            components(dyf, dys);
            float dh2 = 0.0f;
#pragma unroll
            for (int k = 0; k < ODE_S; ++k) dh2 = __builtin_fmaf(w3[k], dys[k], dh2);
            const float da2 = dh2 * (1.0f - h2 * h2);
            const float da1 = rows_sum(row_dot(w2c, da2, 0.0f)) * (1.0f - h1 * h1);
            const float gx = X.sum(turn, L, row_sum2(w1a * da1, w1b * da1, L.lane));
            out[static_cast<uint32_t>(L.unit)] = da1;
            out[static_cast<uint32_t>(ODE_H + L.lane)] = da2;
            out[static_cast<uint32_t>(2 * ODE_H + L.i)] = dyf;  // (the record's last word is a pad)
            return static_cast<double>(gx);
        };
        for (int f = frames - 1; f >= 1; --f) {
            const double next = take(f - 1);  // needed after this frame's substeps
            for (int s = substeps - 1; s >= 0; --s) {
                double dz = lam, dk1 = (h / 6.0) * lam, dk2 = (h / 3.0) * lam, dk3 = (h / 3.0) * lam;
                double gx = vjp((h / 6.0) * lam);
                dz += gx;
                dk3 += h * gx;
                gx = vjp(dk3);
                dz += gx;
                dk2 += 0.5 * h * gx;
                gx = vjp(dk2);
                dz += gx;
                dk1 += 0.5 * h * gx;
                gx = vjp(dk1);
                lam = dz + gx;
            }
            lam += next;
        }
    }
    if (L.w == 0 && (L.lane & 7) == 0 && comp) dz0[L.i] = static_cast<float>(lam);
}

// Parameter gradient from the recorded evaluations (x, h1, h2 in acts; da1,
// da2, dy in adj): dW1 = sum da1 x^T, db1 = sum da1, dW2 = sum da2 h1^T,
// db2 = sum da2, dW3 = sum dy h2^T, db3 = sum dy.  Thread p of chunk c sums
// parameter p over the evaluations [c chunk, (c + 1) chunk) in order; the
// chunks are then added in order, so the result is reproducible.
__global__ __launch_bounds__(256) void k_ode_grad_part(const float* __restrict__ acts, const float* __restrict__ adj,
                                                       int64_t evals, int64_t chunk, float* __restrict__ part) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= N_THETA) return;
    const int64_t e0 = blockIdx.y * chunk;
    const int64_t e1 = e0 + chunk < evals ? e0 + chunk : evals;
    // parameter p as (cotangent index in adj, activation index in acts or -1)
    int ia, ix;
    if (p < OFF_B1) ia = p / 8, ix = p % 8;                                          // W1[j][k]
    else if (p < OFF_W2) ia = p - OFF_B1, ix = -1;                                   // b1[j]
    else if (p < OFF_B2) ia = ODE_H + (p - OFF_W2) / ODE_H, ix = 8 + (p - OFF_W2) % ODE_H;  // W2[j][k]
    else if (p < OFF_W3) ia = ODE_H + (p - OFF_B2), ix = -1;                         // b2[j]
    else if (p < OFF_B3) ia = 2 * ODE_H + (p - OFF_W3) / ODE_H, ix = 8 + ODE_H + (p - OFF_W3) % ODE_H;  // W3[i][j]
    else ia = 2 * ODE_H + (p - OFF_B3), ix = -1;                                     // b3[i]
    float acc = 0.0f;
    for (int64_t e = e0; e < e1; ++e) {
        const float g = adj[e * ODE_ADJ + ia];
        acc = ix >= 0 ? __builtin_fmaf(g, acts[e * ODE_REC + ix], acc) : acc + g;
    }
    part[blockIdx.y * static_cast<int64_t>(N_THETA) + p] = acc;
}

__global__ __launch_bounds__(256) void k_ode_grad_final(const float* __restrict__ part, int64_t chunks,
                                                        float* __restrict__ dtheta) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= N_THETA) return;
    float acc = 0.0f;
#pragma unroll 16
    for (int64_t c = 0; c < chunks; ++c) acc += part[c * N_THETA + p];
    dtheta[p] = acc;
}

// Trajectory error of a camera path against a reference pose table (the
// per-frame poses judging the learned camera of Sec. 3.4).  Per frame, in
// FP64: the camera centre c = -R(q)^T t of each pose and the distance between
// the two centres; the rotation error is the angle of the relative rotation
// R(q) R(q_ref)^T, taken from the relative quaternion q (x) conj(q_ref) as
// 2 atan2(|vector part|, |scalar part|) (both quaternions normalised first).
// One workgroup; the two sums are reduced in a fixed order.
constexpr int PE_WG = 256;

__device__ __forceinline__ void pose_centre(const float* p, double qn[4], double c[3]) {
    double q[4] = {p[0], p[1], p[2], p[3]};
    const double r = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    for (int k = 0; k < 4; ++k) qn[k] = q[k] / r;
    const double w = qn[0], x = qn[1], y = qn[2], z = qn[3];
    const double R[3][3] = {{1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)},
                            {2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)},
                            {2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)}};
    for (int i = 0; i < 3; ++i) c[i] = -(R[0][i] * p[4] + R[1][i] * p[5] + R[2][i] * p[6]);
}

__global__ __launch_bounds__(PE_WG) void k_pose_error(const float* __restrict__ poses, const float* __restrict__ ref,
                                                      int32_t frames, float* __restrict__ per_frame,
                                                      float* __restrict__ summary) {
    __shared__ double s_t[PE_WG], s_a[PE_WG];
    double st = 0.0, sa = 0.0;
    for (int f = threadIdx.x; f < frames; f += PE_WG) {
        double q1[4], c1[3], q2[4], c2[3];
        pose_centre(poses + 7 * f, q1, c1);
        pose_centre(ref + 7 * f, q2, c2);
        const double dx = c1[0] - c2[0], dy = c1[1] - c2[1], dz = c1[2] - c2[2];
        const double te = sqrt(dx * dx + dy * dy + dz * dz);
        // relative quaternion q1 (x) conj(q2)
        const double w = q1[0] * q2[0] + q1[1] * q2[1] + q1[2] * q2[2] + q1[3] * q2[3];
        const double vx = q2[0] * q1[1] - q1[0] * q2[1] - (q1[2] * q2[3] - q1[3] * q2[2]);
        const double vy = q2[0] * q1[2] - q1[0] * q2[2] - (q1[3] * q2[1] - q1[1] * q2[3]);
        const double vz = q2[0] * q1[3] - q1[0] * q2[3] - (q1[1] * q2[2] - q1[2] * q2[1]);
        const double ang = 2.0 * atan2(sqrt(vx * vx + vy * vy + vz * vz), fabs(w));
        per_frame[2 * f] = static_cast<float>(te);
        per_frame[2 * f + 1] = static_cast<float>(ang);
        st += te * te;
        sa += ang;
    }
    s_t[threadIdx.x] = st;
    s_a[threadIdx.x] = sa;
    __syncthreads();
    for (int h = PE_WG / 2; h > 0; h >>= 1) {
        if (static_cast<int>(threadIdx.x) < h) {
            s_t[threadIdx.x] += s_t[threadIdx.x + h];
            s_a[threadIdx.x] += s_a[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        summary[0] = static_cast<float>(sqrt(s_t[0] / frames));
        summary[1] = static_cast<float>(s_a[0] / frames);
    }
}

}  // namespace gv

using namespace gv;

extern "C" {

gv_status gv_camera_ode_workspace_bytes(int32_t frames, int32_t substeps, size_t* out) {
    if (frames < 1 || frames > 100000 || substeps < 1 || substeps > 64 || !out) return GV_ERR_INVALID_ARG;
    *out = ode_layout(frames, substeps).total;
    return GV_OK;
}

gv_status gv_camera_ode_fwd(const float* theta, const float* z0, int32_t frames, int32_t substeps, float* poses,
                            void* ws, size_t ws_bytes, void* stream) {
    if (!theta || !z0 || !poses || frames < 1 || frames > 100000 || substeps < 1 || substeps > 64)
        return GV_ERR_INVALID_ARG;
    const OdeLayout L = ode_layout(frames, substeps);
    if (!ws || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255u)) return GV_ERR_WORKSPACE;
    char* b = static_cast<char*>(ws);
    hipLaunchKernelGGL(k_ode_fwd, dim3(1), dim3(ODE_WG), 0, static_cast<hipStream_t>(stream), theta, z0, frames, substeps,
                       poses, reinterpret_cast<float*>(b + L.acts), reinterpret_cast<double*>(b + L.zf));
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GV_OK : GV_ERR_HIP;
}

gv_status gv_camera_ode_bwd(const float* theta, const float* z0, int32_t frames, int32_t substeps,
                            const float* dL_dposes, float* dtheta, float* dz0, void* ws, size_t ws_bytes,
                            void* stream) {
    if (!theta || !z0 || !dL_dposes || !dtheta || !dz0 || frames < 1 || frames > 100000 || substeps < 1 ||
        substeps > 64)
        return GV_ERR_INVALID_ARG;
    const OdeLayout L = ode_layout(frames, substeps);
    if (!ws || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255u)) return GV_ERR_WORKSPACE;
    char* b = static_cast<char*>(ws);
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const float* acts = reinterpret_cast<const float*>(b + L.acts);
    float* adj = reinterpret_cast<float*>(b + L.adj);
    float* part = reinterpret_cast<float*>(b + L.part);
    hipLaunchKernelGGL(k_ode_bwd, dim3(1), dim3(ODE_WG), 0, st, theta, frames, substeps, dL_dposes, acts,
                       reinterpret_cast<const double*>(b + L.zf), adj, dz0);
    const dim3 pg((N_THETA + 255) / 256, static_cast<uint32_t>(L.chunks));
    hipLaunchKernelGGL(k_ode_grad_part, pg, dim3(256), 0, st, acts, adj, static_cast<int64_t>(L.evals),
                       static_cast<int64_t>(L.chunk), part);
    hipLaunchKernelGGL(k_ode_grad_final, dim3((N_THETA + 255) / 256), dim3(256), 0, st, part,
                       static_cast<int64_t>(L.chunks), dtheta);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GV_OK : GV_ERR_HIP;
}

gv_status gv_pose_error(const float* poses, const float* ref_poses, int32_t frames, float* per_frame, float* summary,
                        void* stream) {
    if (!poses || !ref_poses || !per_frame || !summary || frames < 1 || frames > 100000) return GV_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_pose_error, dim3(1), dim3(PE_WG), 0, static_cast<hipStream_t>(stream), poses, ref_poses,
                       frames, per_frame, summary);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GV_OK : GV_ERR_HIP;
}

}  // extern "C"
