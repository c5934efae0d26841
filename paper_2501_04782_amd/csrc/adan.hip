// Fused Adan step (the optimizer of Sec. 4.1) over several FP32 tensors in
// one launch, reading the parameter, its gradient and the four state words
// (m, v, n, previous gradient) and writing all but the gradient back.
// HBM-bound: per element 24 B read and 20 B written.  A workgroup takes 1,024
// elements of one tensor, a thread four: in a row, with 16-byte accesses, where
// the tensor's pointers and length allow it (a multiple of four elements, so
// that every state row is aligned), else 256 apart.  With one element a thread
// and the tensor found by each element 63 us for 5.6 M elements, 49 us so
// (repeated, their 246 MB stay in the last-level cache; behind 1 GB of other
// traffic 73 and 58 us; 22.4 M elements 251 and 195).
#include <cstring>

#include "gv_internal.h"

namespace gv {

struct AdanTensors {
    float* params[GV_ADAN_MAX_TENSORS];
    const float* grads[GV_ADAN_MAX_TENSORS];
    float* states[GV_ADAN_MAX_TENSORS];      // [4][count]: m, v, n, g_prev
    int64_t counts[GV_ADAN_MAX_TENSORS];
    uint32_t blocks[GV_ADAN_MAX_TENSORS + 1];  // workgroups of the tensors before
    bool wide[GV_ADAN_MAX_TENSORS];            // 16-byte accesses
    int n;
};

constexpr int ADAN_BLOCK = 1024;  // elements

__device__ __forceinline__ void adan_element(const gv_adan_params& hp, float g, float& p, float& m, float& v, float& nn,
                                             float& gp) {
    if (hp.step == 0) {  // m0 = g0, v0 = 0, n0 = g0^2
        m = g;
        v = 0.0f;
        nn = g * g;
    } else {
        const float diff = g - gp;
        m = (1.0f - hp.beta1) * m + hp.beta1 * g;
        v = hp.step == 1 ? diff : (1.0f - hp.beta2) * v + hp.beta2 * diff;  // v1 = g1 - g0
        const float w = g + (1.0f - hp.beta2) * diff;
        nn = (1.0f - hp.beta3) * nn + hp.beta3 * w * w;
    }
    gp = g;
    const float eta = hp.lr / sqrtf(nn + hp.eps);
    p = (p - eta * (m + (1.0f - hp.beta2) * v)) / (1.0f + hp.weight_decay * hp.lr);
}

__global__ __launch_bounds__(256) void k_adan(AdanTensors T, gv_adan_params hp) {
    int t = 0;
    while (t + 1 < T.n && blockIdx.x >= T.blocks[t + 1]) ++t;
    const int64_t c = T.counts[t], j0 = static_cast<int64_t>(blockIdx.x - T.blocks[t]) * ADAN_BLOCK;
    float* ps = T.params[t];
    const float* gs = T.grads[t];
    float* st = T.states[t];
    if (T.wide[t]) {
        const int64_t j = j0 + 4 * threadIdx.x;
        if (j >= c) return;
        auto at = [](float* p) { return reinterpret_cast<float4*>(p); };
        const float4 g = *reinterpret_cast<const float4*>(gs + j);
        float4 p = *at(ps + j), m = {}, v = {}, n = {}, gp = {};
        if (hp.step != 0) {  // the first step's state holds nothing
            m = *at(st + j);
            v = *at(st + c + j);
            n = *at(st + 2 * c + j);
            gp = *at(st + 3 * c + j);
        }
        adan_element(hp, g.x, p.x, m.x, v.x, n.x, gp.x);
        adan_element(hp, g.y, p.y, m.y, v.y, n.y, gp.y);
        adan_element(hp, g.z, p.z, m.z, v.z, n.z, gp.z);
        adan_element(hp, g.w, p.w, m.w, v.w, n.w, gp.w);
        *at(st + j) = m;
        *at(st + c + j) = v;
        *at(st + 2 * c + j) = n;
        *at(st + 3 * c + j) = gp;
        *at(ps + j) = p;
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t j = j0 + 256 * k + threadIdx.x;
        if (j >= c) return;
        float p = ps[j], m = 0.0f, v = 0.0f, n = 0.0f, gp = 0.0f;
        if (hp.step != 0) {
            m = st[j];
            v = st[c + j];
            n = st[2 * c + j];
            gp = st[3 * c + j];
        }
        adan_element(hp, gs[j], p, m, v, n, gp);
        st[j] = m;
        st[c + j] = v;
        st[2 * c + j] = n;
        st[3 * c + j] = gp;
        ps[j] = p;
    }
}

}  // namespace gv

using namespace gv;

extern "C" gv_status gv_adan_step(int32_t n_tensors, float* const* params, const float* const* grads,
                                  float* const* states, const int64_t* counts, const gv_adan_params* hp,
                                  void* stream) {
    if (n_tensors < 1 || n_tensors > GV_ADAN_MAX_TENSORS || !params || !grads || !states || !counts || !hp)
        return GV_ERR_INVALID_ARG;
    if (hp->step < 0 || !(hp->lr >= 0.0f) || !(hp->eps > 0.0f) || !(hp->weight_decay >= 0.0f)) return GV_ERR_INVALID_ARG;
    const float b[3] = {hp->beta1, hp->beta2, hp->beta3};
    for (float x : b)
        if (!(x >= 0.0f && x <= 1.0f)) return GV_ERR_INVALID_ARG;
    AdanTensors T;
    memset(&T, 0, sizeof(T));
    T.n = n_tensors;
    int64_t total = 0, blocks = 0;
    for (int t = 0; t < n_tensors; ++t) {
        if (counts[t] < 0 || (counts[t] > 0 && (!params[t] || !grads[t] || !states[t]))) return GV_ERR_INVALID_ARG;
        T.params[t] = params[t];
        T.grads[t] = grads[t];
        T.states[t] = states[t];
        T.counts[t] = counts[t];
        const uintptr_t bits = reinterpret_cast<uintptr_t>(params[t]) | reinterpret_cast<uintptr_t>(grads[t]) |
                               reinterpret_cast<uintptr_t>(states[t]);
        T.wide[t] = (bits & 15u) == 0u && counts[t] % 4 == 0;
        if (counts[t] > (int64_t(1) << 40) - total) return GV_ERR_INVALID_ARG;
        total += counts[t];
        blocks += (counts[t] + ADAN_BLOCK - 1) / ADAN_BLOCK;
        T.blocks[t + 1] = static_cast<uint32_t>(blocks);
    }
    if (total == 0) return GV_OK;
    hipLaunchKernelGGL(k_adan, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, static_cast<hipStream_t>(stream), T,
                       *hp);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GV_OK : GV_ERR_HIP;
}
