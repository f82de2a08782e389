// Gathered reduced product from K-major activations for problems with too
// few 256 x 256 tiles to fill the chip (Sec. 3.2 definition of RMM; Sec. 3.3
// projections):  Y[b][m][n] = sum_{t < k} Xt[b][I_b[t]][m] * W[I_b[t]][n].
//
// The same data path as the large-tile kernel (gemm.hip): the retained rows
// of Xt and W go straight into an LDS ring by 16-byte buffer loads, S - 1
// stages ahead, and come back as MFMA fragments through the transposing LDS
// read; Y^T tiles, so a lane ends with four consecutive n of one m.  What
// bounds these sizes is the number of CUs at work and the length of the
// dependent K loop, so the tiles are smaller:
//   128 x 128 (eight waves of 64 x 32, 32-row stages, 78 KiB of LDS: two
//     workgroups per CU) from about 256 tiles of 64 x 64 up to the sizes the
//     256 x 256 tile fills;
//   64 x 64 (four waves of 32 x 32, 64-row stages: half as many barriers) up
//     to there.
// Each output is one chain of MFMAs over the list in order, as in the other
// bf16 kernels, so all of them give the same bits (four waves that split the
// K loop of a 64 x 64 tile, added at the end, were no faster: 12.5 us for the
// first shape below).
// The retained list is read from LDS (segments of kMidSeg indices, copied by
// the whole workgroup), because a staged row here is shorter than 512 bytes
// and one load instruction covers 4 or 8 rows with a different index each.
//
// Measured against the register-staged 128 x 128 kernel these replace (us,
// bf16): 37 x 4096 -> 6144 at r = 0.5 38.0 -> 11.3, 16 x 14336 -> 4096 at
// r = 0.5 118 -> 33, 777 x 4096 -> 4096 at r = 0.8 63.8 -> 32 to 34 (610 to
// 650 TFLOP/s), 2048 x 8192 -> 2048 at r = 0.5 77 -> 40 (850 TFLOP/s); and
// against the 256 x 256 tile where that leaves half the chip idle, 2048 x 4096
// -> 4096 at r = 0.5 48.5 -> 37.4.  Also timed, no better (with a barrier that
// did not yet wait for the LDS reads, 31.0 us for the third shape): four waves
// of 64 x 64, 64-row stages, three slots (31-48 us for the third shape); 256 x
// 128 and 128 x 256 tiles (43-48); 64 x 128 (42); for 64 x 64, 32- or 128-row
// stages (12.2-13.9 us for the first shape), tiles 32 wide (12.7-19).
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rmm {

namespace {

constexpr int kMidSeg = 3584;      // retained indices held in LDS at a time (14 KiB: two workgroups per CU)

template <int N>
__device__ __forceinline__ void mid_wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// A 16-lane group of the transposing read takes 32 bytes of four consecutive
// staged rows, its neighbour the next 32: the 64-byte block q of row r is
// stored at q ^ mid_swz(r), so that those four rows fall on distinct banks.
template <int ROWB>
__device__ __forceinline__ int mid_swz(int r) {
    return ROWB >= 256 ? (r & 3) : ROWB == 128 ? ((r >> 1) & 1) : 0;
}

// WM x WN waves cover a BM x BN tile, BKS retained rows per stage.  Units u
// read weights W + (u / w_ugroup) * w_ustride.  trim: X is zero at (m, j) for
// j > m + trim_off, and the K loop stops at the tile's last row's limit; with
// a one-dimensional grid the units then go round fastest and the tiles with
// the longest loops first, so that the short ones fill the tail (32 heads x
// 4096 causal queries, 2048 kept tokens: 67 us; 107 with 256 x 128 tiles).
template <int BM, int BN, int WM, int WN, int BKS, int S>
__global__ __launch_bounds__(WM *WN * 64, WM *WN / 4) void gemm_kmajor_mid_kernel(
    const uint16_t *__restrict__ Xt, const uint16_t *__restrict__ W, const int32_t *__restrict__ idx,
    uint16_t *__restrict__ Y, int B, int M, int N, int k, int64_t ldxt, int64_t ldw, int64_t ldy,
    int64_t xt_bytes, int64_t w_bytes, int tiles_m, int tiles_n, int vec_y, int64_t w_ustride,
    int w_ugroup, int trim, int64_t trim_off) {
    constexpr int NW = WM * WN, NT = NW * 64;
    constexpr int RA = BM * 2, RB = BN * 2;             // bytes per staged row
    constexpr int ASZ = BKS * RA, BSZ = BKS * RB;
    constexpr int PA = ASZ / 1024 / NW, PB = BSZ / 1024 / NW;   // DMA instructions per wave per stage
    constexpr int LPA = RA / 16, LPB = RB / 16;         // lanes per staged row
    constexpr int RPA = 64 / LPA, RPB = 64 / LPB;       // rows per instruction
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int D = S - 1, PER = PA + PB;
    static_assert(PA >= 1 && PB >= 1 && PA * NW * 1024 == ASZ && PB * NW * 1024 == BSZ, "staging split");
    static_assert(BKS % 16 == 0 && FM >= 1 && FN >= 1 && S >= 2 && S <= 4, "layout");
    static_assert((D - 1) * PER < 64, "vmcnt range");
    __shared__ __attribute__((aligned(1024))) char sA0[ASZ], sA1[ASZ], sA2[S > 2 ? ASZ : 16], sA3[S > 3 ? ASZ : 16];
    __shared__ __attribute__((aligned(1024))) char sB0[BSZ], sB1[BSZ], sB2[S > 2 ? BSZ : 16], sB3[S > 3 ? BSZ : 16];
    __shared__ __attribute__((aligned(16))) int32_t il[kMidSeg];
    auto stage_a = [&](auto I) -> char * {
        constexpr int i = decltype(I)::value;
        if constexpr (i == 0) return sA0;
        else if constexpr (i == 1) return sA1;
        else if constexpr (i == 2) return sA2;
        else return sA3;
    };
    auto stage_b = [&](auto I) -> char * {
        constexpr int i = decltype(I)::value;
        if constexpr (i == 0) return sB0;
        else if constexpr (i == 1) return sB1;
        else if constexpr (i == 2) return sB2;
        else return sB3;
    };

    const int T = tiles_m * tiles_n;
    const int bid = static_cast<int>(blockIdx.x);
    int unit, tm, tn;
    if (trim && gridDim.y == 1) {
        unit = bid % B;
        const int rank = bid / B;
        tm = tiles_m - 1 - rank / tiles_n;
        tn = rank % tiles_n;
    } else {
        unit = static_cast<int>(blockIdx.y);
        // the 8 XCDs take workgroups in turn: a contiguous run of tiles each,
        // four tile rows at a time, so that its L2 serves the shared panels
        const int lin = (T % 8 == 0) ? (bid % 8) * (T / 8) + bid / 8 : bid;
        constexpr int GM = 4;
        const int gsz = GM * tiles_n;
        const int first_m = (lin / gsz) * GM;
        const int gm = min(GM, tiles_m - first_m);
        tm = first_m + (lin % gsz) % gm;
        tn = (lin % gsz) / gm;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t *I = idx + static_cast<int64_t>(unit) * k;
    int kk = k;
    if (trim) {                                  // I is ascending: a binary search
        const int64_t jmax = static_cast<int64_t>(m0) + BM - 1 + trim_off;
        int lo = 0, hi = k;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (static_cast<int64_t>(I[mid]) <= jmax) lo = mid + 1; else hi = mid;
        }
        kk = __builtin_amdgcn_readfirstlane(lo);
    }

    constexpr uint32_t kOut = 0x80000000u;
    const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(Xt + unit * (xt_bytes / 2)), 0, static_cast<uint32_t>(xt_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(W + (unit / w_ugroup) * w_ustride), 0, static_cast<uint32_t>(w_bytes), 0x00020000);
    const uint32_t arow = static_cast<uint32_t>(ldxt) * 2u, brow = static_cast<uint32_t>(ldw) * 2u;

    // DMA role: instruction e of the wave fills 1 KiB = RPA (RPB) staged rows,
    // a lane one 16-byte chunk of row lane / LPA.  Rows past the list read out
    // of range and stage zeros; columns past M or N read neighbouring data
    // that only reaches outputs never stored.
    const int ra = lane / LPA, rb = lane / LPB;
    uint32_t acol[PA], bcol[PB];
#pragma unroll
    for (int e = 0; e < PA; ++e)
        acol[e] = static_cast<uint32_t>(m0 + 8 * ((lane % LPA) ^ (4 * mid_swz<RA>((RPA * (wave * PA + e) + ra) & 3)))) * 2u;
#pragma unroll
    for (int e = 0; e < PB; ++e)
        bcol[e] = static_cast<uint32_t>(n0 + 8 * ((lane % LPB) ^ (4 * mid_swz<RB>((RPB * (wave * PB + e) + rb) & 3)))) * 2u;

    // fragment role: as in the large-tile kernel
    const int wm = wave / WN, wn = wave % WN;
    const int g = lane >> 4, s16 = lane & 15, f4 = (s16 >> 2) & 3;
    const int rowl = 8 * (g >> 1) + (s16 >> 2);
    const int coll = 32 * (g & 1) + 8 * (s16 & 3);
    int aoff[FM], boff[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) aoff[i] = rowl * RA + coll + 64 * ((wm * FM + i) ^ mid_swz<RA>(f4));
#pragma unroll
    for (int j = 0; j < FN; ++j) boff[j] = rowl * RB + coll + 64 * ((wn * FN + j) ^ mid_swz<RB>(f4));
    auto frag = [&](const char *base, auto R) -> bf16x8_t {
        constexpr int rowb = decltype(R)::value;
        const s16x4_t lo = lds_read_tr16(base);
        const s16x4_t hi = lds_read_tr16(base + 4 * rowb);
        typedef short s16x8_t __attribute__((ext_vector_type(8)));
        const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8_t, v);
    };

    f32x16_t acc[FN][FM];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;

    // a barrier that does not wait for the loads still landing in LDS, only for
    // this wave's own LDS reads: the slot they read is refilled by the other
    // waves right after it.  Every step issues one stage of loads (past the
    // end: zeros), so the vmcnt wait before it is a fixed count.
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    auto barrier = []() {
        __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
        asm volatile("s_barrier" ::: "memory");
    };

    for (int seg = 0; seg < kk; seg += kMidSeg) {
        const int ks_n = min(kMidSeg, kk - seg);
        if (seg > 0) __syncthreads();
        for (int t = tid; t < ks_n; t += NT) il[t] = I[seg + t];
        __syncthreads();
        const int nT = (ks_n + BKS - 1) / BKS;
        int32_t ja[PA], jb[PB];
        auto fetch = [&](int st) {
#pragma unroll
            for (int e = 0; e < PA; ++e) ja[e] = il[min(st * BKS + RPA * (wave * PA + e) + ra, kMidSeg - 1)];
            if constexpr (BM != BN) {
#pragma unroll
                for (int e = 0; e < PB; ++e) jb[e] = il[min(st * BKS + RPB * (wave * PB + e) + rb, kMidSeg - 1)];
            }
        };
        auto dma = [&](auto slot, int st) {
            char *la = stage_a(slot), *lb = stage_b(slot);
#pragma unroll
            for (int e = 0; e < PA; ++e) {
                const bool in = st * BKS + RPA * (wave * PA + e) + ra < ks_n;
                lds_load16(ar, la + (wave * PA + e) * 1024, in ? static_cast<uint32_t>(ja[e]) * arow + acol[e] : kOut);
            }
#pragma unroll
            for (int e = 0; e < PB; ++e) {
                const bool in = st * BKS + RPB * (wave * PB + e) + rb < ks_n;
                const int32_t j = BM == BN ? ja[e % PA] : jb[e];
                lds_load16(br, lb + (wave * PB + e) * 1024, in ? static_cast<uint32_t>(j) * brow + bcol[e] : kOut);
            }
        };
        auto prologue = [&](auto Iv) {
            constexpr int st = decltype(Iv)::value;
            if constexpr (st < D) { fetch(st); dma(Iv, st); }
        };
        prologue(I0{});
        prologue(I1{});
        prologue(I2{});
        fetch(D);
        mid_wait_vmcnt<(D - 1) * PER>();
        barrier();
        auto step = [&](auto Iv, int t) {
            constexpr int slot = decltype(Iv)::value;
            dma(std::integral_constant<int, (slot + D) % S>{}, t + D);
            fetch(t + D + 1);
            const char *la = stage_a(Iv), *lb = stage_b(Iv);
#pragma unroll
            for (int ks = 0; ks < BKS / 16; ++ks) {
                bf16x8_t a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = frag(la + aoff[i] + ks * 16 * RA, std::integral_constant<int, RA>{});
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = frag(lb + boff[j] + ks * 16 * RB, std::integral_constant<int, RB>{});
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
                        acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[j][i], 0, 0, 0);
            }
            mid_wait_vmcnt<(D - 1) * PER>();
            barrier();
        };
        int t0 = 0;
        for (; t0 + S <= nT; t0 += S) {
            step(I0{}, t0);
            step(I1{}, t0 + 1);
            if constexpr (S > 2) step(I2{}, t0 + 2);
            if constexpr (S > 3) step(I3{}, t0 + 3);
        }
        if (t0 < nT) step(I0{}, t0);
        if constexpr (S > 2) { if (t0 + 1 < nT) step(I1{}, t0 + 1); }
        if constexpr (S > 3) { if (t0 + 2 < nT) step(I2{}, t0 + 2); }
        mid_wait_vmcnt<0>();
    }

    // acc[j][i][4*gq + r]: n = n0 + wn*TN + 32j + 8gq + 4*(lane/32) + r,
    //                      m = m0 + wm*TM + 32i + lane%32
    const int lr = lane & 31, lh = lane >> 5;
    uint16_t *Yt = Y + (static_cast<int64_t>(unit) * M + m0) * ldy;
    const int rows = min(BM, M - m0);
    if constexpr (BM == 64) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int ml = wm * TM + 32 * i + lr;
                    const int n = n0 + wn * TN + 32 * j + 8 * gq + 4 * lh;
                    if (ml >= rows) continue;
                    const uint32_t w0 = pack_bf16x2(acc[j][i][4 * gq], acc[j][i][4 * gq + 1]);
                    const uint32_t w1 = pack_bf16x2(acc[j][i][4 * gq + 2], acc[j][i][4 * gq + 3]);
                    uint16_t *p = Yt + ml * ldy + n;
                    if (vec_y && n + 4 <= N) {
                        *reinterpret_cast<uint2 *>(p) = make_uint2(w0, w1);
                    } else {
                        const uint16_t e[4] = {static_cast<uint16_t>(w0), static_cast<uint16_t>(w0 >> 16),
                                               static_cast<uint16_t>(w1), static_cast<uint16_t>(w1 >> 16)};
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr)
                            if (n + rr < N) p[rr] = e[rr];
                    }
                }
        return;
    }
    // Through the idle ring, so that neighbouring lanes write neighbouring
    // pieces of a row (16, 8 or 2 bytes, as Y's rows are aligned; where the tile
    // is cut by N too): OR rows per X slot, 16-byte chunk c of a row at c ^ (row %
    // CH).  Against pieces of four elements straight from the accumulators (us): 5820
    // x 72 -> 352, k = 36 9.4 -> 5.4, 602 x 72 -> 3565 (odd) 11.2 -> 6.9, 2536 x 1024 -> 1864
    // in rows of 1867, k = 768 30 -> 19.
    constexpr int CH = BN / 8, OR = ASZ / RB;
    static_assert(BM == 64 || (OR % 32 == 0 && BM == S * OR), "staged output");
    auto obj = [&](int r) -> char * {
        const int q = r / OR;
        return (q == 0 ? sA0 : q == 1 ? sA1 : q == 2 ? sA2 : sA3) + (r % OR) * RB;
    };
    __syncthreads();                                     // every wave's last reads and loads are done
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const int r = wm * TM + 32 * i + lr, c = (wn * TN) / 8 + 4 * j + gq;
                *reinterpret_cast<uint2 *>(obj(r) + 16 * (c ^ (r % CH)) + 8 * lh) =
                    make_uint2(pack_bf16x2(acc[j][i][4 * gq], acc[j][i][4 * gq + 1]),
                               pack_bf16x2(acc[j][i][4 * gq + 2], acc[j][i][4 * gq + 3]));
            }
    __syncthreads();
    // elements n .. n + U - 1 of row r, per thread
    auto out = [&](auto Uv) {
        constexpr int U = decltype(Uv)::value, LPR = BN / U, RPP = NT / LPR;
        const int u = tid % LPR, n = n0 + U * u;
#pragma unroll
        for (int p = 0; p < BM / RPP; ++p) {
            const int r = RPP * p + tid / LPR;
            if (r >= rows) continue;
            const char *src = obj(r) + 16 * ((U * u / 8) ^ (r % CH)) + 2 * (U * u % 8);
            uint16_t *dst = Yt + r * ldy + n;
            if (n + U <= N) {
                if constexpr (U == 8) *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src);
                else if constexpr (U == 4) *reinterpret_cast<uint2 *>(dst) = *reinterpret_cast<const uint2 *>(src);
                else *dst = *reinterpret_cast<const uint16_t *>(src);
            } else if constexpr (U > 1) {
#pragma unroll
                for (int e = 0; e < U - 1; ++e)
                    if (n + e < N) dst[e] = reinterpret_cast<const uint16_t *>(src)[e];
            }
        }
    };
    if (vec_y == 2) out(std::integral_constant<int, 8>{});
    else if (vec_y == 1) out(std::integral_constant<int, 4>{});
    else out(std::integral_constant<int, 1>{});
}

template <int BM, int BN, int WM, int WN, int BKS, int S>
hipError_t launch_mid(const uint16_t *Xt, const uint16_t *W, const int32_t *idx, int64_t B, int64_t M,
                      int64_t N, int64_t K, int64_t k, int64_t ldxt, int64_t ldw, uint16_t *Y, int64_t ldy,
                      int64_t w_ustride, int w_ugroup, int trim, int64_t trim_off, hipStream_t stream) {
    const int vec_y = (reinterpret_cast<uintptr_t>(Y) % 16 == 0 && ldy % 8 == 0) ? 2
                      : (reinterpret_cast<uintptr_t>(Y) % 8 == 0 && ldy % 4 == 0) ? 1 : 0;
    const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    const bool flat = trim && tm * tn * B <= (1 << 22);
    const dim3 grid(static_cast<unsigned>(flat ? tm * tn * B : tm * tn), static_cast<unsigned>(flat ? 1 : B));
    hipLaunchKernelGGL((gemm_kmajor_mid_kernel<BM, BN, WM, WN, BKS, S>), grid, dim3(WM * WN * 64), 0,
                       stream, Xt, W, idx, Y, static_cast<int>(B), static_cast<int>(M), static_cast<int>(N),
                       static_cast<int>(k), ldxt, ldw, ldy, K * ldxt * 2, K * ldw * 2, static_cast<int>(tm),
                       static_cast<int>(tn), vec_y, w_ustride, w_ugroup, trim, trim_off);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_kmajor_mid_bf16(bool wide, const uint16_t *Xt, const uint16_t *W, const int32_t *idx,
                                       int64_t B, int64_t M, int64_t N, int64_t K, int64_t k, int64_t ldxt,
                                       int64_t ldw, uint16_t *Y, int64_t ldy, int64_t w_ustride, int w_ugroup,
                                       int trim, int64_t trim_off, hipStream_t stream) {
    return wide ? launch_mid<128, 128, 2, 4, 32, 4>(Xt, W, idx, B, M, N, K, k, ldxt, ldw, Y, ldy, w_ustride,
                                                       w_ugroup, trim, trim_off, stream)
                : launch_mid<64, 64, 2, 2, 64, 4>(Xt, W, idx, B, M, N, K, k, ldxt, ldw, Y, ldy, w_ustride,
                                                     w_ugroup, trim, trim_off, stream);
}

}  // namespace rmm
