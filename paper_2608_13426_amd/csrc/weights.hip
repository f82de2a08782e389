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
// 16 or 64 lanes per query row read the row's kept scores once (with the causal
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

// f over the LANES (16 or 64) lanes of a row group (every lane ends with the same value)
template <int LANES, typename F>
__device__ __forceinline__ float across(float x, F f) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto step = [&](auto ctrl) {
        x = f(x, __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
                     0, static_cast<int>(__float_as_uint(x)), decltype(ctrl)::value, 0xF, 0xF, false))));
    };
    step(std::integral_constant<int, 0xB1>{});           // lane ^ 1
    step(std::integral_constant<int, 0x4E>{});           // lane ^ 2
    step(std::integral_constant<int, 0x141>{});          // mirror within 8
    step(std::integral_constant<int, 0x140>{});          // mirror within 16
    if constexpr (LANES == 64) {
        x = f(x, __shfl_xor(x, 16));
        x = f(x, __shfl_xor(x, 32));
    }
#endif
    return x;
}

// LANES (16, or a wave) per query row, eight 16-byte loads in flight each.  Per
// lane a running maximum over its 64-key batches in order and a sum rescaled
// when the maximum rises; then the lanes' maxima, and their rescaled sums in a
// fixed tree.  32 heads x 2048 causal rows: 49.5 -> 39.3 us (a wave per row, two
// loads per lane on average, a merge with two exponentials at each of six steps).
// Chunks that no lane of the wave has are passed over, and only the chunk that a
// row's limit falls into is masked: 8 heads x 40 causal rows 13.2 -> 8.4 us for
// the whole call, against a mask and eight exponentials for each of eight chunks.
template <int LANES>
__global__ __launch_bounds__(kRowThreads) void softmax_rowstats_kernel(
    const uint16_t *__restrict__ S, int64_t U, int64_t Lq, int64_t Lk, int64_t lds, int causal,
    float *__restrict__ rmax, float *__restrict__ rinv) {
    const int sub = threadIdx.x % LANES;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * (kRowThreads / LANES) + threadIdx.x / LANES;
    const bool live = row < U * Lq;                      // every lane stays for the row groups' moves
    const int64_t i = live ? row % Lq : 0;
    const uint16_t *s = S + (live ? row : 0) * lds;      // units are packed: unit stride Lq * lds
    // keys 0 .. nk-1 are kept (the causal mask keeps t <= i + Lk - Lq); Lk < 2^31
    const int nk = static_cast<int>(!live ? 0 : causal ? max<int64_t>(0, min<int64_t>(Lk, i + Lk - Lq + 1)) : Lk);
    const int nc = nk / 8 + (nk % 8 != 0);
    float m = -INFINITY;
    double l = 0.0;
    for (int c0 = sub; c0 < nc; c0 += 8 * LANES) {
        uint4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + LANES * u;
            q[u] = c < nc ? *reinterpret_cast<const uint4 *>(s + 8 * static_cast<int64_t>(c))
                          : make_uint4(0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u);   // -inf
        }
        // chunks in the wave: the first lane of a row group has the most
        int nu = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) nu += __builtin_amdgcn_ballot_w64(c0 + LANES * u < nc) != 0;
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (u >= nu) break;
            uint32_t *w = reinterpret_cast<uint32_t *>(&q[u]);
            if (c0 + LANES * u == nc - 1 && nk % 8 != 0) {   // keys past the row's limit count as -inf
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (2 * e >= nk % 8) w[e] = (w[e] & 0xffff0000u) | 0xff80u;
                    if (2 * e + 1 >= nk % 8) w[e] = (w[e] & 0xffffu) | 0xff800000u;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                cm = fmaxf(cm, fmaxf(__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xffff0000u)));
        }
        if (cm == -INFINITY) continue;                   // every key of the batch masked
        if (cm > m) {
            l = m == -INFINITY ? 0.0 : l * static_cast<double>(__expf(m - cm));
            m = cm;
        }
        float l8[8] = {};                                // chains of up to eight, then float64
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (u >= nu) break;
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
    const float mm = across<LANES>(m, [](float a, float b) { return fmaxf(a, b); });
    l = m == -INFINITY ? 0.0 : l * static_cast<double>(__expf(m - mm));
    l += dpp_f64<0xB1>(l);
    l += dpp_f64<0x4E>(l);
    l += dpp_f64<0x141>(l);
    l += dpp_f64<0x140>(l);
    if constexpr (LANES == 64) {
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
    }
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
    const int64_t rows = U * Lq;
    auto stats = [&](auto kernel, int64_t per) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((rows + per - 1) / per)), dim3(kRowThreads), 0, stream,
                           S, U, Lq, Lk, lds, causal, rmax, rinv);
    };
    // A wave per row where 16 lanes would make the chain of a row's batches long
    // for the number of rows that hide it.  The whole call in us, 64 / 16 lanes:
    // 200 rows x 1000 keys 8.9 / 9.6, 4000 x 1000 15.5 / 15.0; 4000 x 2048 22.8 / 25.5,
    // 16000 x 2048 43.1 / 45.1, 32000 x 1504 60.7 / 56.3; 32000 x 4096 equal, x 8192
    // 424 / 438; 200 x 8192 13.0 / 24.2.
    if (Lk >= 4096 || (rows <= 16384 && Lk >= 2048) || (rows <= 2048 && Lk > 512))
        stats(softmax_rowstats_kernel<64>, kRowThreads / 64);
    else stats(softmax_rowstats_kernel<16>, kRowThreads / 16);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_score_softmax_kmajor(S, U, Lq, Lk, lds, rmax, rinv, Lk - Lq, causal, energy, partials,
                                       Pt, ldpt, stream);
}

}  // namespace rmm
