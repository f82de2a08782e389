// Attention weights P = softmax(S + M) written K-major with their token
// energies (Sec. 3.3: the token scores of the value product are the column
// norms of P; the Limitations section names the memory movement of a
// separate scoring pass as a cost to remove).
//
//   rmax[i]   = max over kept t of S[i][t],  rsum[i] = sum over kept t of
//               exp(S[i][t] - rmax[i])                         (fp32)
//   Pt[t][i]  = bf16(exp(S[i][t] - rmax[i]) / rsum[i]), 0 where masked
//   energy[t] = sum over i of Pt[t][i]^2                       (float64)
//
// Two launches, as for the normalisation producer.  softmax_rowstats_kernel:
// 16 lanes per query row read the row's kept scores once (with the causal
// mask, only the keys up to the row's limit: the masked half of S is never
// read), keeping a running maximum and a sum rescaled whenever the maximum
// rises, per lane in key order and then merged across the lanes in a fixed
// tree.  Then the scoring pass's
// transposing tile kernel in its softmax variant forms the weights in
// registers and writes them K-major as whole 128-byte row segments with the
// float64 column energies; its wave tiles that lie wholly above the causal
// diagonal read nothing and write zeros.
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rmm {

namespace {

constexpr int kRowThreads = 256;
constexpr int kRowLanes = 16;                            // lanes per row
constexpr int kRowsPerBlock = kRowThreads / kRowLanes;

// f over the 16 lanes of a row group (every lane ends with the same value)
template <typename F>
__device__ __forceinline__ float across16(float x, F f) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto step = [&](auto ctrl) {
        x = f(x, __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
                     0, static_cast<int>(__float_as_uint(x)), decltype(ctrl)::value, 0xF, 0xF, false))));
    };
    step(std::integral_constant<int, 0xB1>{});           // lane ^ 1
    step(std::integral_constant<int, 0x4E>{});           // lane ^ 2
    step(std::integral_constant<int, 0x141>{});          // mirror within 8
    step(std::integral_constant<int, 0x140>{});          // mirror within 16
#endif
    return x;
}

// 16 lanes per query row, eight 16-byte loads in flight each.  Per lane a
// running maximum over its 64-key batches in order and a sum rescaled when the
// maximum rises; then the lanes' maxima, and their rescaled sums in a fixed
// tree.  32 heads x 2048 causal rows: 49.5 -> 39.3 us (a wave per row, two loads
// per lane on average, a merge with two exponentials at each of six steps).
__global__ __launch_bounds__(kRowThreads) void softmax_rowstats_kernel(
    const uint16_t *__restrict__ S, int64_t U, int64_t Lq, int64_t Lk, int64_t lds, int causal,
    float *__restrict__ rmax, float *__restrict__ rinv) {
    const int sub = threadIdx.x % kRowLanes;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * kRowsPerBlock + threadIdx.x / kRowLanes;
    const bool live = row < U * Lq;                      // every lane stays for the row groups' moves
    const int64_t i = live ? row % Lq : 0;
    const uint16_t *s = S + (live ? row : 0) * lds;      // units are packed: unit stride Lq * lds
    // keys 0 .. nk-1 are kept (the causal mask keeps t <= i + Lk - Lq)
    const int64_t nk = !live ? 0 : causal ? max<int64_t>(0, min<int64_t>(Lk, i + Lk - Lq + 1)) : Lk;
    const int64_t nc = (nk + 7) / 8;
    float m = -INFINITY;
    double l = 0.0;
    for (int64_t c0 = sub; c0 < nc; c0 += 8 * kRowLanes) {
        uint4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t c = c0 + kRowLanes * u;
            q[u] = c < nc ? *reinterpret_cast<const uint4 *>(s + 8 * c)
                          : make_uint4(0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u);   // -inf
        }
        if (8 * (c0 + 7 * kRowLanes) + 8 > nk) {         // keys past the row's limit count as -inf
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t left = nk - 8 * (c0 + kRowLanes * u);
                uint32_t *w = reinterpret_cast<uint32_t *>(&q[u]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (2 * e >= left) w[e] = (w[e] & 0xffff0000u) | 0xff80u;
                    if (2 * e + 1 >= left) w[e] = (w[e] & 0xffffu) | 0xff800000u;
                }
            }
        }
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t w[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                cm = fmaxf(cm, fmaxf(__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xffff0000u)));
        }
        if (cm == -INFINITY) continue;                   // every key of the batch masked
        if (cm > m) {
            l = m == -INFINITY ? 0.0 : l * static_cast<double>(__expf(m - cm));
            m = cm;
        }
        float l8[8] = {};                                // chains of eight, then float64
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t w[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                l8[2 * e] += __expf(__uint_as_float(w[e] << 16) - m);     // exp(-inf) = 0
                l8[2 * e + 1] += __expf(__uint_as_float(w[e] & 0xffff0000u) - m);
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) l += static_cast<double>(l8[e]);
    }
    const float mm = across16(m, [](float a, float b) { return fmaxf(a, b); });
    l = m == -INFINITY ? 0.0 : l * static_cast<double>(__expf(m - mm));
    l += dpp_f64<0xB1>(l);
    l += dpp_f64<0x4E>(l);
    l += dpp_f64<0x141>(l);
    l += dpp_f64<0x140>(l);
    if (live && sub == 0) {
        const bool empty = !(l > 0.0);
        rmax[row] = empty ? 0.f : mm;
        rinv[row] = empty ? 0.f : static_cast<float>(1.0 / l);
    }
}

inline size_t align256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

}  // namespace

size_t weights_workspace_bytes(int64_t U, int64_t Lq, int64_t Lk) {
    return 2 * align256(static_cast<size_t>(U * Lq) * sizeof(float)) + score_workspace_bytes(U, Lq, Lk);
}

hipError_t launch_attention_weights_kmajor(const uint16_t *S, int64_t U, int64_t Lq, int64_t Lk,
                                           int64_t lds, int causal, const float *rmax_in,
                                           const float *rinv_in, uint16_t *Pt, int64_t ldpt,
                                           double *energy, void *workspace, hipStream_t stream) {
    char *ws = static_cast<char *>(workspace);
    float *rmax = reinterpret_cast<float *>(ws);
    float *rinv = reinterpret_cast<float *>(ws + align256(static_cast<size_t>(U * Lq) * sizeof(float)));
    double *partials = reinterpret_cast<double *>(ws + 2 * align256(static_cast<size_t>(U * Lq) * sizeof(float)));
    if (rmax_in && rinv_in)
        return launch_score_softmax_kmajor(S, U, Lq, Lk, lds, rmax_in, rinv_in, Lk - Lq, causal, energy,
                                           partials, Pt, ldpt, stream);
    const int64_t rows = U * Lq, per = kRowsPerBlock;
    hipLaunchKernelGGL(softmax_rowstats_kernel, dim3(static_cast<unsigned>((rows + per - 1) / per)),
                       dim3(kRowThreads), 0, stream, S, U, Lq, Lk, lds, causal, rmax, rinv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_score_softmax_kmajor(S, U, Lq, Lk, lds, rmax, rinv, Lk - Lq, causal, energy, partials,
                                       Pt, ldpt, stream);
}

}  // namespace rmm
