// Reduced attention block for a few query rows per head (a decode step, or a
// handful of tokens against a long cache):
//   O[q] = softmax(scale * Q[q][I_h] . K[t][I_h]) V,  one set I_h per query head.
//
// Bound by reading K and V once: 2 * Lk * 256 bytes per (sequence, kv head).
// The prefill kernel (attn.hip) gives each query head one workgroup that walks
// all keys, after a pass that writes every head's compacted keys: at 8
// sequences x 32 heads x 4001 keys that is 256 workgroups with 1 of 256 query
// rows in use and a compaction of 2.5 times the bytes of K and V.  Here
//   * nothing is compacted: whole key rows are staged in LDS and each head's
//     wave clears the dims outside I_h in its fragments (bitwise, so that an
//     infinite or NaN key value outside the set stays without effect), against
//     a query fragment with the same dims cleared; up to 16 query rows are the
//     16 columns of v_mfma_f32_16x16x32_bf16;
//   * the query heads of one kv head share each staged tile: GH heads x KS
//     tiles of 32 keys are the waves of a workgroup;
//   * the keys are split over S workgroups, enough to keep every CU loading;
//     each writes its maximum, weight sum and unnormalised fp32 output, which a
//     second kernel merges in split order (S = 1 writes O).
// Scores, softmax and the weights' rounding are those of the prefill kernel
// (fp32 scores in log2 units, weights rounded to bf16 for the value product).
//
// Measured against the prefill kernel (us, one query row, 64 of 128 dims, K and
// V from a rotating set): 8 sequences x 32 heads on 8 kv heads x 4001 keys 154
// -> 31 (4.3 TB/s of K and V), one sequence 90 -> 15, with 16384 keys 328 -> 28,
// 32 sequences x 2000 keys 279 -> 53 (5.0 TB/s), 4 x 32 kv heads x 4000 keys 115
// -> 53 (5.0 TB/s).
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rmm {

namespace {

namespace fewk {
constexpr int D = 128, ROWB = D * 2;       // head dim, bytes per key / value row
constexpr int TQ = 16;                     // query rows per workgroup
constexpr int TS = 32;                     // keys per wave and stage
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kTau = 8.f;                // lazy-rescale threshold, log2 units
// Workgroups aimed at: two per CU where four or eight heads share a workgroup.
// One and two heads take 131 and 99 KB of LDS, so one workgroup per CU, and 512
// of them are two rounds.
constexpr int kBlocks = 512;
constexpr int kMinTiles = 4;               // stages per split at least
constexpr int kFewMaxRows = 256;           // query rows per head taken here at most

template <int N>
__device__ __forceinline__ void wait_vmcnt_le() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// f over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (all of them get the result)
template <typename F>
__device__ __forceinline__ float across_rows(float x, F f) {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = f(__uint_as_float(b[0]), __uint_as_float(b[1]));
#endif
    return x;
}
}  // namespace fewk

// One workgroup: query rows q0 .. q0+15 of heads h0 .. h0+GH-1 (of one kv
// head), stages [s * tps, (s + 1) * tps) of KS * 32 keys; NS ring slots.
template <int GH, int KS, int NS>
__global__ __launch_bounds__(GH *KS * 64) void attn_few_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ V,
    const int32_t *__restrict__ idx, uint16_t *__restrict__ O, float *__restrict__ part, int H, int Hkv,
    int Lq, int Lk, int k, float c, int neg_q, int causal, int S, int tps, int64_t rows_total, int direct) {
    using namespace fewk;
    constexpr int NW = GH * KS, NT = NW * 64;
    constexpr int TK = TS * KS, KB = TK * ROWB;         // keys and bytes of K (or V) per stage
    constexpr int PER_K = KB / 1024 / NW, PER = 2 * PER_K;   // DMA instructions per wave per stage
    constexpr int DA = NS - 1;
    static_assert(PER_K >= 1 && PER_K * NW * 1024 == KB && NS >= 2 && NS <= 4, "staging split");
    __shared__ __attribute__((aligned(1024))) char sl0[2 * KB], sl1[2 * KB], sl2[NS > 2 ? 2 * KB : 16],
        sl3[NS > 3 ? 2 * KB : 16];
    __shared__ __attribute__((aligned(16))) uint16_t keep[GH][D];    // 0xffff at the head's retained dims
    auto slot_at = [&](auto I) -> char * {
        constexpr int i = decltype(I)::value;
        if constexpr (i == 0) return sl0;
        else if constexpr (i == 1) return sl1;
        else if constexpr (i == 2) return sl2;
        else return sl3;
    };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hw = wave % GH, kw = wave / GH;           // head of the chunk, key tile of the stage
    const int col = lane & 15, g = lane >> 4;           // query row (MFMA column), lane group
    const int grp = H / Hkv, hch = (grp + GH - 1) / GH, nqb = (Lq + TQ - 1) / TQ;
    int w = static_cast<int>(blockIdx.x);
    const int s = w % S; w /= S;
    const int q0 = (w % nqb) * TQ; w /= nqb;
    const int hc = w % hch; w /= hch;
    const int gk = w % Hkv, b = w / Hkv;
    const int h = gk * grp + hc * GH + hw;
    const bool head_ok = hc * GH + hw < grp;            // wave-uniform
    const int64_t bh = static_cast<int64_t>(b) * H + (head_ok ? h : gk * grp);

    const uint16_t *Kh = Kc + (static_cast<int64_t>(b) * Hkv + gk) * Lk * D;
    const uint16_t *Vh = V + (static_cast<int64_t>(b) * Hkv + gk) * Lk * D;
    // no row of the block keeps a key at or past kend: those are staged as zeros
    // (a masked key's weight is zero, but 0 * infinity is not), whole tiles skipped
    const int kend = causal ? max(0, min(Lk, min(q0 + TQ, Lq) + Lk - Lq)) : Lk;
    const int n_tiles = (kend + TK - 1) / TK;
    const int t_begin = s * tps, t_end = min(n_tiles, t_begin + tps);

    // DMA role: instruction u of the wave fills rows 4j .. 4j+3 of the stage,
    // j = wave + NW * u.  Key chunk p of row r sits at p ^ (r % 16): eight rows
    // at one chunk are eight bank groups.  A value row's 32-byte unit u sits at
    // u ^ (r % 8): the eight rows that two 16-lane groups of a transposing read
    // take together are eight units.
    uint32_t ksrc[PER_K], vsrc[PER_K];
#pragma unroll
    for (int u = 0; u < PER_K; ++u) {
        const int r = 4 * (wave + NW * u) + (lane >> 4), p = lane & 15;
        ksrc[u] = static_cast<uint32_t>(r * ROWB + 16 * (p ^ (r & 15)));
        vsrc[u] = static_cast<uint32_t>(r * ROWB + 32 * ((p >> 1) ^ (r & 7)) + 16 * (p & 1));
    }
    auto dma = [&](char *slot, int t) __attribute__((always_inline)) {
        // tiles past the split's end read nothing and stage zeros
        const int t0 = __builtin_amdgcn_readfirstlane(min(t * TK, kend));
        const int rows = __builtin_amdgcn_readfirstlane(t < t_end ? min(TK, kend - t0) : 0);
        const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(Kh + static_cast<int64_t>(t0) * D), 0, static_cast<uint32_t>(rows * ROWB), 0x00020000);
        const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(Vh + static_cast<int64_t>(t0) * D), 0, static_cast<uint32_t>(rows * ROWB), 0x00020000);
#pragma unroll
        for (int u = 0; u < PER_K; ++u) lds_load16(kr, slot + 1024 * (wave + NW * u), ksrc[u]);
#pragma unroll
        for (int u = 0; u < PER_K; ++u) lds_load16(vr, slot + KB + 1024 * (wave + NW * u), vsrc[u]);
    };

    // query rows and the head's list, then the first stages (loads return in
    // order: waiting for the former leaves the latter in flight)
    uint4 qraw[D / 32];
    int32_t jl[D / 64];
    {
        const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(Q + (bh * Lq + q0) * D), 0, static_cast<uint32_t>(min(TQ, Lq - q0) * ROWB), 0x00020000);
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b128(qr, static_cast<uint32_t>(col * ROWB + 64 * ks + 16 * g), 0, 0);
            qraw[ks] = make_uint4(x[0], x[1], x[2], x[3]);
        }
#pragma unroll
        for (int u = 0; u < D / 64; ++u) jl[u] = idx[bh * k + min(lane + 64 * u, k - 1)];
    }
    dma(sl0, t_begin);
    if constexpr (DA > 1) dma(sl1, t_begin + 1);
    if constexpr (DA > 2) dma(sl2, t_begin + 2);

    // the head's retained dims and its masked query fragments
    for (int i = tid; i < GH * D / 8; i += NT) reinterpret_cast<uint4 *>(&keep[0][0])[i] = make_uint4(0, 0, 0, 0);
    lds_barrier();
    if (kw == 0) {
#pragma unroll
        for (int u = 0; u < D / 64; ++u) keep[hw][jl[u]] = 0xffffu;
    }
    lds_barrier();
    bf16x8_t qf[D / 32];
    uint4 km[D / 32];
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) {
        km[ks] = *reinterpret_cast<const uint4 *>(&keep[hw][32 * ks + 8 * g]);
        const uint32_t flip = neg_q ? 0x80008000u : 0u;       // exact negation, for scale < 0
        qf[ks] = __builtin_bit_cast(bf16x8_t, make_uint4((qraw[ks].x ^ flip) & km[ks].x, (qraw[ks].y ^ flip) & km[ks].y,
                                                         (qraw[ks].z ^ flip) & km[ks].z, (qraw[ks].w ^ flip) & km[ks].w));
    }

    // per-lane fragment addresses within a stage
    const int krow = TS * kw + col;                     // key row (+ 16 for the second half)
    int voff[D / 16];
    {
        const int r = TS * kw + 4 * g + ((lane & 15) >> 2);
#pragma unroll
        for (int db = 0; db < D / 16; ++db) voff[db] = KB + r * ROWB + 32 * (db ^ (r & 7)) + 8 * (lane & 3);
    }

    f32x4_t o[D / 16];
#pragma unroll
    for (int db = 0; db < D / 16; ++db) o[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = -__builtin_inff(), l_run = 0.f;
    // this lane's query keeps keys <= lim
    const int lim = causal ? min(q0 + col + Lk - Lq, Lk - 1) : Lk - 1;

    auto tile = [&](const char *slot, int t) __attribute__((always_inline)) {
        const int t0 = t * TK + TS * kw;
        if (t0 >= kend) return;                         // wave-uniform
        f32x4_t sc[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            sc[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            const int r = krow + 16 * tb;
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks) {
                const uint4 x = *reinterpret_cast<const uint4 *>(slot + r * ROWB + 16 * ((4 * ks + g) ^ (r & 15)));
                const bf16x8_t kf = __builtin_bit_cast(
                    bf16x8_t, make_uint4(x.x & km[ks].x, x.y & km[ks].y, x.z & km[ks].z, x.w & km[ks].w));
                sc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[ks], sc[tb], 0, 0, 0);
            }
        }
        // sc[tb][r]: key t0 + 16*tb + 4*g + r of query row col
        const int rel = lim - t0 - 4 * g;
        float mx = -__builtin_inff();
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (16 * tb + r > rel) sc[tb][r] = -__builtin_inff();
                mx = fmaxf(mx, sc[tb][r]);
            }
        mx = across_rows(mx, [](float a, float e) { return fmaxf(a, e); });
        const float mt = mx == -__builtin_inff() ? -__builtin_inff() : mx * c;
        const bool need = mt > m_run + kTau;
        if (__builtin_amdgcn_ballot_w64(need)) {
            const float alpha = need ? __builtin_amdgcn_exp2f(m_run - mt) : 1.f;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < D / 16; ++db) o[db] *= alpha;
            m_run = need ? mt : m_run;
        }
        // a row with nothing kept yet has only masked (-inf) scores here
        const float mu = m_run == -__builtin_inff() ? 0.f : m_run;
        bf16x8_t pf;                                     // slot e: key 16*(e/4) + 4*g + e%4
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e >> 2][e & 3], c, -mu));
            l_run += p;
            pf[e] = static_cast<__bf16>(p);
        }
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const s16x4_t lo = lds_read_tr16(slot + voff[db]);
            const s16x4_t hi = lds_read_tr16(slot + voff[db] + 16 * ROWB);
            const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[db], 0, 0, 0);
        }
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    // every step issues one stage of loads, so the wait before each barrier is fixed
    auto step = [&](auto Iv, int t) __attribute__((always_inline)) {
        constexpr int sl = decltype(Iv)::value;
        wait_vmcnt_le<(DA - 1) * PER>();
        lds_barrier();                                   // stage t landed; the slot read last step is free
        dma(slot_at(std::integral_constant<int, (sl + DA) % NS>{}), t + DA);
        tile(slot_at(Iv), t);
    };
    for (int t = t_begin; t < t_end; t += NS) {
        step(I0{}, t);
        if (t + 1 < t_end) step(I1{}, t + 1);
        if constexpr (NS > 2) { if (t + 2 < t_end) step(I2{}, t + 2); }
        if constexpr (NS > 3) { if (t + 3 < t_end) step(I3{}, t + 3); }
    }
    wait_vmcnt_le<0>();                                  // the trailing loads
    float l = across_rows(l_run, [](float a, float e) { return a + e; });

    if constexpr (KS > 1) {
        // the other key tiles' waves hand over (m, l, o), merged in tile order
        constexpr int WB = 64 * 16 * (D / 16) + 64 * 8;
        static_assert((KS - 1) * GH * WB <= 2 * KB, "merge area");
        __syncthreads();
        if (kw > 0) {
            char *p = sl0 + ((kw - 1) * GH + hw) * WB;
#pragma unroll
            for (int db = 0; db < D / 16; ++db) *reinterpret_cast<f32x4_t *>(p + 1024 * db + 16 * lane) = o[db];
            *reinterpret_cast<float2 *>(p + 1024 * (D / 16) + 8 * lane) = make_float2(m_run, l);
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int j = 0; j < KS - 1; ++j) {
            const char *p = sl0 + (j * GH + hw) * WB;
            const float2 ml = *reinterpret_cast<const float2 *>(p + 1024 * (D / 16) + 8 * lane);
            const float mm = fmaxf(m_run, ml.x);
            const float fa = m_run == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(m_run - mm);
            const float fb = ml.x == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(ml.x - mm);
            l = l * fa + ml.y * fb;
            m_run = mm;
#pragma unroll
            for (int db = 0; db < D / 16; ++db)
                o[db] = o[db] * fa + *reinterpret_cast<const f32x4_t *>(p + 1024 * db + 16 * lane) * fb;
        }
    }
    if (!head_ok || q0 + col >= Lq) return;
    const int64_t row = bh * Lq + q0 + col;
    if (direct) {                                        // one split
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int db = 0; db < D / 16; ++db)
            *reinterpret_cast<uint2 *>(O + row * D + 16 * db + 4 * g) =
                make_uint2(pack_bf16x2(o[db][0] * inv, o[db][1] * inv), pack_bf16x2(o[db][2] * inv, o[db][3] * inv));
        return;
    }
    float *po = part + (row * S + s) * D;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) *reinterpret_cast<f32x4_t *>(po + 16 * db + 4 * g) = o[db];
    if (g == 0) *reinterpret_cast<float2 *>(part + rows_total * S * D + (row * S + s) * 2) = make_float2(m_run, l);
}

// dims d (and, with W = 2, d + 1) of a row: the splits' outputs merged in split order
template <int W>
__device__ __forceinline__ void merge_row(const float *__restrict__ part, int64_t rows, int64_t row, int S, int d,
                                          float (&out)[W]) {
    const float2 *ml = reinterpret_cast<const float2 *>(part + rows * S * fewk::D) + row * S;
    const float *po = part + row * S * fewk::D + d;
    float m = -__builtin_inff();
    for (int s = 0; s < S; ++s) m = fmaxf(m, ml[s].x);
    float l = 0.f, a[W] = {};
#pragma unroll 4
    for (int s = 0; s < S; ++s) {
        const float2 x = ml[s];
        const float f = x.x == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(x.x - m);
        l += x.y * f;
#pragma unroll
        for (int w = 0; w < W; ++w) a[w] += po[s * fewk::D + w] * f;
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) out[w] = a[w] * inv;
}

// O[row][d]: a wave per row, two dims per lane
__global__ __launch_bounds__(256) void attn_few_merge_kernel(const float *__restrict__ part,
                                                             uint16_t *__restrict__ O, int64_t rows, int S) {
    const int lane = threadIdx.x & 63;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    float v[2];
    merge_row(part, rows, row, S, 2 * lane, v);
    reinterpret_cast<uint32_t *>(O)[row * (fewk::D / 2) + lane] = pack_bf16x2(v[0], v[1]);
}

// Ot[bh*D + d][q] and its energies, the queries in order: a thread per dim of one
// head walks the rows, without LDS or barriers (the same conditions as below)
__global__ __launch_bounds__(fewk::D) void attn_few_merge_dims_kernel(
    const float *__restrict__ part, uint16_t *__restrict__ Ot, int64_t ldot, double *__restrict__ energy, int Lq,
    int S, int64_t rows) {
    const int64_t bh = blockIdx.x, row_t = bh * fewk::D + threadIdx.x;
    double e = 0.0;
    for (int q0 = 0; q0 < Lq; q0 += 8) {
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float v[1];
            merge_row(part, rows, bh * Lq + q0 + q, S, static_cast<int>(threadIdx.x), v);
            const uint32_t x = f32_to_bf16(v[0]);
            const double y = static_cast<double>(__uint_as_float(x << 16));
            e = fma(y, y, e);
            w[q >> 1] = q & 1 ? w[q >> 1] | (x << 16) : x;
        }
        *reinterpret_cast<uint4 *>(Ot + row_t * ldot + q0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    energy[row_t] = e;
}

// Ot[bh*D + d][q] and its energies for DIMS dims of one head (blockIdx.x): a
// thread merges one dim of a row at a time, up to ROWS rows at once, through LDS into
// rows of Ot; the energies are added over the queries in a fixed order (Lq % 8 ==
// 0, Lq <= MAXR, rows of Ot 16-byte aligned).  32 heads on 8 kv heads x 4000 keys,
// the whole call in us with 16 dims, 8 / 64 / 256 rows: 17 / 28 / 59 (a thread per dim
// walking all rows 38 / 163 / 293, the prefill kernel 93 / 94 / 95).  Many heads need
// no such split, and fewer, larger workgroups take less (the rule below).
template <int DIMS, int ROWS, int MAXR>
__global__ __launch_bounds__(ROWS *DIMS) void attn_few_merge_kmajor_kernel(
    const float *__restrict__ part, uint16_t *__restrict__ Ot, int64_t ldot, double *__restrict__ energy, int Lq,
    int S, int64_t rows) {
    constexpr int LR = MAXR + 8;                               // staged dim row (16-byte aligned)
    __shared__ __attribute__((aligned(16))) uint16_t val[DIMS][LR];
    __shared__ double en[DIMS][MAXR / 8];
    const int tid = threadIdx.x, nt = blockDim.x, d0 = DIMS * static_cast<int>(blockIdx.x);
    const int64_t bh = blockIdx.y;
    for (int q = tid / DIMS; q < Lq; q += nt / DIMS) {
        float v[1];
        merge_row(part, rows, bh * Lq + q, S, d0 + tid % DIMS, v);
        val[tid % DIMS][q] = f32_to_bf16(v[0]);
    }
    __syncthreads();
    const int nq = Lq / 8;
    for (int i = tid; i < DIMS * nq; i += nt) {
        const int d = i / nq, c = i % nq;
        const uint4 x = *reinterpret_cast<const uint4 *>(&val[d][8 * c]);
        *reinterpret_cast<uint4 *>(Ot + (bh * fewk::D + d0 + d) * ldot + 8 * c) = x;
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
        double e = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double y0 = static_cast<double>(__uint_as_float(w[j] << 16));
            const double y1 = static_cast<double>(__uint_as_float(w[j] & 0xffff0000u));
            e = fma(y0, y0, e);
            e = fma(y1, y1, e);
        }
        en[d][c] = e;
    }
    __syncthreads();
    if (tid < DIMS) {
        double e = 0.0;
        for (int c = 0; c < nq; ++c) e += en[tid][c];
        energy[bh * fewk::D + d0 + tid] = e;
    }
}

}  // namespace

namespace {

// query heads of one kv head that share a workgroup
int head_chunk(int64_t grp) { return grp == 1 ? 1 : grp == 2 ? 2 : grp <= 4 ? 4 : 8; }

// The splits' launch (O null: partials also for one split); *S_out splits.
hipError_t launch_splits(const uint16_t *Q, const uint16_t *Kc, const uint16_t *V, const int32_t *idx,
                                int64_t batch, int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk, int64_t k,
                                float scale, bool causal, uint16_t *O, float *part, int *S_out,
                                hipStream_t stream) {
    using namespace fewk;
    const int64_t grp = H / Hkv;
    const int gh = head_chunk(grp);
    const int64_t tk = TS * (gh == 1 ? 4 : gh == 2 ? 2 : 1);
    const int64_t tiles = (Lk + tk - 1) / tk;
    const int64_t base = batch * Hkv * ((grp + gh - 1) / gh) * ((Lq + TQ - 1) / TQ);
    int64_t S = (kBlocks + base - 1) / base;
    if (S > tiles / kMinTiles) S = tiles / kMinTiles;
    const int64_t rows = batch * H * Lq;
    const int64_t fit = static_cast<int64_t>(attn_workspace_bytes(batch * H, Lk, k) /
                                             (static_cast<size_t>(rows) * (D + 2) * sizeof(float)));
    if (S > fit) S = fit;
    if (S < 1) S = 1;
    const int64_t tps = (tiles + S - 1) / S;
    S = (tiles + tps - 1) / tps;
    // |scale| in log2 units; a zero scale as the smallest normal float (see the
    // prefill kernel's launcher)
    float c = (scale < 0.f ? -scale : scale) * kLog2e;
    if (c < 1.17549435e-38f) c = 1.17549435e-38f;
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(base * S)), dim3(threads), 0, stream, Q, Kc, V, idx, O,
                           part, static_cast<int>(H), static_cast<int>(Hkv),
                           static_cast<int>(Lq), static_cast<int>(Lk), static_cast<int>(k), c, scale < 0.f ? 1 : 0,
                           causal ? 1 : 0, static_cast<int>(S), static_cast<int>(tps), rows, O && S == 1 ? 1 : 0);
    };
    if (gh == 1) launch(attn_few_kernel<1, 4, 2>, 256);
    else if (gh == 2) launch(attn_few_kernel<2, 2, 3>, 256);
    else if (gh == 4) launch(attn_few_kernel<4, 1, 4>, 256);
    else launch(attn_few_kernel<8, 1, 4>, 512);
    *S_out = static_cast<int>(S);
    return hipGetLastError();
}

}  // namespace

// Which calls come here.  One split's partials must fit the workspace (Lk * kp
// * 2 bytes per head), which keeps prefills (Lk close to Lq) out.  Up to 16 rows
// always: K and V pass once.  Above, each 16 rows pass them again, from L2 at
// about 6.5 TB/s (512 bytes per key and 16-row block of a head chunk), while
// the prefill kernel takes 22.5 ns per key and round of 256 workgroups: the
// former is shorter below 285 such blocks per round (us, 4000 keys: 2 sequences
// x 32 heads x 64 rows, 256 blocks, 80 against 101; 128 rows, 512 blocks, 144
// against 102; 4 x 32 heads on 8 kv heads x 128 rows, 256 blocks, 69 against 116).
bool attn_few_ok(int64_t batch, int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk, int64_t k) {
    if (Lq > fewk::kFewMaxRows || Lk * attn_k_steps(k) * 32 < Lq * (fewk::D + 2) * static_cast<int64_t>(sizeof(float))) return false;
    if (Lq <= fewk::TQ) return true;
    const int64_t grp = H / Hkv, chunk = head_chunk(grp);
    const int64_t blocks = batch * Hkv * ((grp + chunk - 1) / chunk) * ((Lq + fewk::TQ - 1) / fewk::TQ);
    return blocks < 285 * ((batch * H + 255) / 256);
}

hipError_t launch_attn_few_bf16(const uint16_t *Q, const uint16_t *Kc, const uint16_t *V, const int32_t *idx,
                                int64_t batch, int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk, int64_t k,
                                float scale, bool causal, uint16_t *O, void *workspace, hipStream_t stream) {
    int S = 1;
    float *part = static_cast<float *>(workspace);
    const hipError_t e = launch_splits(Q, Kc, V, idx, batch, H, Hkv, Lq, Lk, k, scale, causal, O, part, &S, stream);
    if (e != hipSuccess || S == 1) return e;
    const int64_t rows = batch * H * Lq;
    hipLaunchKernelGGL(attn_few_merge_kernel, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, stream,
                       part, O, rows, S);
    return hipGetLastError();
}

hipError_t launch_attn_few_kmajor_bf16(const uint16_t *Q, const uint16_t *Kc, const uint16_t *V,
                                       const int32_t *idx, int64_t batch, int64_t H, int64_t Hkv, int64_t Lq,
                                       int64_t Lk, int64_t k, float scale, bool causal, uint16_t *Ot,
                                       int64_t ldot, double *energy, void *workspace, hipStream_t stream) {
    int S = 1;
    float *part = static_cast<float *>(workspace);
    const hipError_t e = launch_splits(Q, Kc, V, idx, batch, H, Hkv, Lq, Lk, k, scale, causal, nullptr, part, &S, stream);
    if (e != hipSuccess) return e;
    auto merge = [&](auto kern, int dims, int at_once) {
        hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(fewk::D / dims), static_cast<unsigned>(batch * H)),
                           dim3(static_cast<unsigned>(dims * (Lq < at_once ? Lq : at_once))), 0, stream, part, Ot,
                           ldot, energy, static_cast<int>(Lq), S, batch * H * Lq);
    };
    // us, 16 dims / 128 dims / a thread per dim: 512 heads x 8 rows x 64 keys 12.0 / 10.7 /
    // 12.1, 1024 x 8 x 1000 36.6 / 33.5 / 36.1, 1792 x 8 x 64 22.7 / 17.7 / 17.2, 8192 x 8 x 64
    // 67.5 / 51.9 / 45.5, 4096 x 24 x 300 113 / 94.7 / 95.9; 256 x 16 x 300 15.5 / 16.8 / 22.9
    if (Lq > 32 || batch * H < 512) merge(attn_few_merge_kmajor_kernel<16, 32, fewk::kFewMaxRows>, 16, 32);
    else if (batch * H < 1536 || Lq > 16) merge(attn_few_merge_kmajor_kernel<128, 4, 32>, 128, 4);
    else hipLaunchKernelGGL(attn_few_merge_dims_kernel, dim3(static_cast<unsigned>(batch * H)), dim3(fewk::D), 0,
                            stream, part, Ot, ldot, energy, static_cast<int>(Lq), S, batch * H * Lq);
    return hipGetLastError();
}

}  // namespace rmm
