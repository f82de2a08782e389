// Reduced attention scores over head-dim slices (Sec. 3.3, Attention):
//   S[h] = scale * Q[h][:, I_h] K[g(h)][:, I_h]^T,  -inf where causally masked,
// with g(h) = h / (H / Hkv).
//
// A Q row and a K row are each D contiguous values.  The kernels are bound by
// writing S (Lq*Lk values per head), which does not shrink with k; tiles lying
// wholly above the causal diagonal skip the product and only write -inf.  Head
// dims of 64 and 128 take the row-streaming kernel below; other head dims the
// tile kernel, whose operands are gathered at the retained dims.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rmm {

namespace {

constexpr uint16_t kBf16NegInf = 0xff80;

template <int BM, int BN, int BK, int WM, int WN>
__global__ __launch_bounds__(WM *WN *kWave) void qk_bf16_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kc,
    const int32_t *__restrict__ idx, uint16_t *__restrict__ S, int H, int Hkv, int Lq, int Lk,
    int D, int k, float scale, int causal) {
    constexpr int NT = WM * WN * kWave;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int LDS_K = BK + 8;
    constexpr int PASS = NT / BK;
    constexpr int A_PER_T = BM / PASS, B_PER_T = BN / PASS;
    static_assert(NT % BK == 0 && BM % PASS == 0 && BN % PASS == 0, "tile split");

    __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDS_K];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDS_K];

    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int wm = wave / WN, wn = wave % WN;
    const int bh = blockIdx.z, b = bh / H, h = bh % H, g = h / (H / Hkv);
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int off = Lk - Lq;
    const uint16_t *Qh = Q + static_cast<int64_t>(bh) * Lq * D;
    const uint16_t *Kh = Kc + (static_cast<int64_t>(b) * Hkv + g) * Lk * D;
    const int32_t *I = idx + static_cast<int64_t>(bh) * k;
    uint16_t *Sh = S + static_cast<int64_t>(bh) * Lq * Lk;

    if (causal && n0 > m0 + BM - 1 + off) {          // wholly masked tile
        for (int v = tid; v < BM * BN; v += NT) {
            const int m = m0 + v / BN, n = n0 + v % BN;
            if (m < Lq && n < Lk) Sh[static_cast<int64_t>(m) * Lk + n] = kBf16NegInf;
        }
        return;
    }

    const int a_t = tid % BK, row0 = tid / BK;
    uint16_t a_reg[A_PER_T], b_reg[B_PER_T];
    auto fetch = [&](int t0) {
        const int t = t0 + a_t;
        const int j = t < k ? I[t] : -1;
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) {
            const int m = m0 + row0 + i * PASS;
            a_reg[i] = (j >= 0 && m < Lq) ? Qh[static_cast<int64_t>(m) * D + j] : uint16_t(0);
        }
#pragma unroll
        for (int i = 0; i < B_PER_T; ++i) {
            const int n = n0 + row0 + i * PASS;
            b_reg[i] = (j >= 0 && n < Lk) ? Kh[static_cast<int64_t>(n) * D + j] : uint16_t(0);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) As[(row0 + i * PASS) * LDS_K + a_t] = a_reg[i];
#pragma unroll
        for (int i = 0; i < B_PER_T; ++i) Bs[(row0 + i * PASS) * LDS_K + a_t] = b_reg[i];
    };

    f32x16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int lr = lane % 32, lk = (lane / 32) * 8;
    fetch(0);
    for (int t0 = 0; t0 < k; t0 += BK) {
        stash();
        __syncthreads();
        if (t0 + BK < k) fetch(t0 + BK);
#pragma unroll
        for (int ks = 0; ks < BK; ks += 16) {
            bf16x8_t a[FM], bb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i)
                a[i] = *reinterpret_cast<const bf16x8_t *>(&As[(wm * TM + i * 32 + lr) * LDS_K + ks + lk]);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                bb[j] = *reinterpret_cast<const bf16x8_t *>(&Bs[(wn * TN + j * 32 + lr) * LDS_K + ks + lk]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bb[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int n = n0 + wn * TN + j * 32 + lr;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm * TM + i * 32 + 8 * (v / 4) + 4 * (lane / 32) + (v % 4);
                if (m < Lq && n < Lk) {
                    const bool masked = causal && n > m + off;
                    Sh[static_cast<int64_t>(m) * Lk + n] =
                        masked ? kBf16NegInf : f32_to_bf16(acc[i][j][v] * scale);
                }
            }
        }
}

// ------------------------------------------------------- row-streaming kernel
// One workgroup per (head, 128-query tile, share of the key tiles) walks its
// key tiles (BT keys: 128 with 4 waves, or 256 with 8 waves).  Q and K rows (D
// values, 16-byte chunks) are read whole and staged in LDS.
//   Masked (the usual form): the dropped dims are cleared on the way into LDS
//   and the product runs over all D dims, with 16-byte fragment reads.  The
//   matrix work is the same for every k and stays behind the stores.
//   Gathered (GATHER, long rows with few dims): an odd row stride of D/2+1
//   words, so 32 rows read at one column hit 32 distinct banks; the fragments
//   are gathered at the retained dims with 2-byte reads (a zeroed pad word
//   stands in for padding positions).  With few dims kept one strip of 32 keys
//   per wave against all 128 queries, so no K fragment is gathered twice.
// Q's fragments are kept in registers.  The waves split the 128 x BT tile into
// KW key strips and WQ query strips.  The product is formed transposed (keys x
// queries), so each lane holds 4 consecutive keys of one query; tiles are
// staged through LDS and written as coalesced 16-byte stores, BT*2-byte row
// pieces.  Key tiles wholly above the diagonal are streamed as -inf.
// Bound by writing S.  Measured (us, causal, before -> now; gathered fragments,
// no key shares and a 2-byte fallback for odd rows before): 32 heads x 1001 keys,
// k = 103 53.6 -> 18.5; x 1024, k = 64 19.3 -> 15.9; x 4096, k = 64 249 -> 232 (4.6
// TB/s); x 4095 642 -> 331; 8 sequences x 32 heads, one query x 4001 keys 99 -> 45.
namespace rowk {
constexpr int BQ = 128;       // queries per block
// cache policy of the score stores (sc1).  Streaming (nt) stores measured
// about 25% slower for this pattern of 256-byte row pieces 2*Lk bytes apart.
constexpr int kStoreAux = 16;
}  // namespace rowk

// ST: also write each score row's softmax statistics over the stored bf16
// scores of its kept keys: rmax[row] = their maximum, rinv[row] = 1 / sum of
// exp(s - rmax) (0 and 0 for a row with nothing kept).  They are taken where
// the staged tile is read back for its stores: each thread keeps, for each of
// its rows, a running maximum over its 8-key chunks and a sum rescaled when
// the maximum rises; a row's threads are consecutive lanes, merged at the end
// in a fixed butterfly.
// MODE: 0 rows on 16-byte boundaries; 1 any rows (buffer stores need no
// alignment; the chunk a row ends in goes out element by element); 2 any rows,
// shifted to lines: row pieces that do not cover whole 128-byte lines write at
// about 60 % of the rate of those that do, so the pieces start at line
// boundaries and each row's elements past the last one wait for the next tile.
template <int D, int WQ, int NTT, int BTT, bool ST = false, int MODE = 0, bool GATHER = false>
__global__ __launch_bounds__(NTT, NTT == 256 ? 2 : 1) void qk_bf16_rows_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kc,
    const int32_t *__restrict__ idx, uint16_t *__restrict__ S, int H, int Hkv, int Lq, int Lk,
    int k, float scale, int causal, int C, float *__restrict__ rmax = nullptr,
    float *__restrict__ rinv = nullptr) {
    constexpr int BQ = rowk::BQ, BT = BTT, NT = NTT;
    constexpr bool RAG = MODE == 2, ANY = MODE > 0;
    constexpr int PRE = RAG ? 64 : 0;      // the previous tile's last columns before a staged row
    constexpr int OS = PRE + BT + 8;       // staged output row (16-byte aligned)
    typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
    constexpr int kStoreAux = RAG ? 0 : rowk::kStoreAux;
    constexpr int RW = GATHER ? D / 2 + 1 : D / 2;   // words per staged row (odd: 32 rows, 32 banks)
    constexpr int KSMAX = GATHER ? 4 : D / 16;       // k-steps
    constexpr int CH = D / 8;              // 16-byte chunks per row
    constexpr int PER_T = BT * CH / NT;    // chunks staged per thread
    constexpr int KW = NT / 64 / WQ;       // waves along keys
    constexpr int FI = BT / KW / 32;       // 32-key fragments per wave
    constexpr int FJ = BQ / WQ / 32;       // 32-query fragments per wave
    static_assert(D % 16 == 0 && BT % BQ == 0 && (BT * CH) % NT == 0, "shape");
    static_assert((WQ == 1 || WQ == 2) && NT % CH == 0, "shape");

    __shared__ __attribute__((aligned(1024))) uint32_t rows_lds[BT * RW];
    __shared__ __attribute__((aligned(16))) uint16_t out_lds[BQ * OS];
    // masked: 0xffff at the retained dims; gathered: their byte offsets in a row
    __shared__ __attribute__((aligned(16))) uint16_t dims[D + 16];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bh = blockIdx.y, b = bh / H, h = bh % H, g = h / (H / Hkv);
    // causal: the last query tiles carry the most key tiles, so they are
    // dealt first (longest work first keeps the tail of the grid short)
    const int qx = static_cast<int>(blockIdx.x) / C, chunk = static_cast<int>(blockIdx.x) % C;
    const int qt = causal ? static_cast<int>(gridDim.x) / C - 1 - qx : qx;
    const int q0 = qt * BQ;
    const int off = Lk - Lq;
    const int32_t *I = idx + static_cast<int64_t>(bh) * k;
    uint16_t *Sh = S + static_cast<int64_t>(bh) * Lq * Lk;
    const int n_tiles = (Lk + BT - 1) / BT;
    int n_compute = n_tiles;
    if (causal) {
        const int limit = min(q0 + BQ, Lq) - 1 + off;   // largest key any row keeps
        n_compute = limit < 0 ? 0 : min(n_tiles, limit / BT + 1);
    }
    // this block's key tiles: [t_lo, t_hi), the first nc of them with a product
    const int tpc = (n_tiles + C - 1) / C, t_lo = chunk * tpc, t_hi = min(n_tiles, t_lo + tpc);
    const int nc = max(0, min(t_hi, n_compute) - t_lo);
    // Store role: a wave instruction covers RPI row pieces of the tile, CPR
    // 16-byte chunks each; RAG: of rows equal mod 8 (one 16-byte misalignment)
    constexpr int CPR = BT / 8, RPI = 64 / CPR, NWV = NT / 64;
    constexpr int RES = 8 / NWV, SR = BQ / RPI / NWV, IPR = SR / RES;   // residues, instructions (and each) per wave
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int c16 = lane % CPR;
    auto row_of = [&](int i) {
        return RAG ? wave_u + NWV * (i / IPR) + 8 * (RPI * (i % IPR) + lane / CPR) : tid / CPR + RPI * NWV * i;
    };
    // RAG: elements between the last 128-byte boundary of memory and row r
    const int s_mis = RAG ? static_cast<int>((reinterpret_cast<uintptr_t>(Sh + static_cast<int64_t>(q0) * Lk) / 2) & 63) : 0;
    auto mis = [&](int r) { return RAG ? (s_mis + r * Lk) & 63 : 0; };
    // the block's rows of S; rows at or past Lq fall outside the range and are dropped
    const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc(
        Sh + static_cast<int64_t>(q0) * Lk, 0, static_cast<uint32_t>(min(BQ, Lq - q0) * Lk * 2),
        0x00020000);
    float st_m[SR], st_l[SR];                 // their running statistics (ST)
#pragma unroll
    for (int i = 0; i < SR; ++i) { st_m[i] = -__builtin_inff(); st_l[i] = 0.f; }

    if (nc > 0) {
        const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(Q + (static_cast<int64_t>(bh) * Lq + q0) * D), 0,
            static_cast<uint32_t>(min(BQ, Lq - q0) * D * 2), 0x00020000);
        const uint16_t *Kh = Kc + (static_cast<int64_t>(b) * Hkv + g) * Lk * D;

        uint4 regs[PER_T];
        auto load_rows = [&](__amdgpu_buffer_rsrc_t rs) {
#pragma unroll
            for (int i = 0; i < PER_T; ++i) {
                const int v = tid + NT * i;
                const auto x = __builtin_amdgcn_raw_buffer_load_b128(
                    rs, static_cast<uint32_t>(((v / CH) * D + (v % CH) * 8) * 2), 0, 0);
                regs[i] = make_uint4(x[0], x[1], x[2], x[3]);
            }
        };
        // masked: a thread's chunks all lie in one 16-byte column of the rows, so
        // one mask clears the dropped dims on the way into LDS (bitwise: an
        // infinite or NaN value there stays without effect); chunk c of row r
        // sits at c ^ (r % CH)
        const int KS = GATHER ? (k + 15) / 16 : KSMAX;
        uint4 km = make_uint4(0, 0, 0, 0);
        auto store_rows = [&]() {
#pragma unroll
            for (int i = 0; i < PER_T; ++i) {
                const int v = tid + NT * i, r = v / CH;
                if constexpr (GATHER) {
                    uint32_t *dst = rows_lds + r * RW + (v % CH) * 4;
                    dst[0] = regs[i].x; dst[1] = regs[i].y; dst[2] = regs[i].z; dst[3] = regs[i].w;
                } else {
                    *reinterpret_cast<uint4 *>(rows_lds + r * RW + 4 * ((v % CH) ^ (r & (CH - 1)))) =
                        make_uint4(regs[i].x & km.x, regs[i].y & km.y, regs[i].z & km.z, regs[i].w & km.w);
                }
            }
        };
        auto key_rsrc = [&](int kt) {
            const int t0 = kt * BT;
            return __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t *>(Kh + static_cast<int64_t>(t0) * D), 0,
                static_cast<uint32_t>(min(BT, Lk - t0) * D * 2), 0x00020000);
        };
        // 8 dims (k-step ks, lane half) of staged row `row`
        auto frag = [&](int row, int ks) -> bf16x8_t {
            if constexpr (GATHER) {
                const uint4 co = *reinterpret_cast<const uint4 *>(&dims[ks * 16 + 8 * (lane >> 5)]);
                const char *base = reinterpret_cast<const char *>(rows_lds + row * RW);
                const uint32_t o[4] = {co.x, co.y, co.z, co.w};
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t lo = *reinterpret_cast<const uint16_t *>(base + (o[q] & 0xffffu));
                    const uint32_t hi = *reinterpret_cast<const uint16_t *>(base + (o[q] >> 16));
                    w[q] = lo | (hi << 16);
                }
                return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
            } else {
                return *reinterpret_cast<const bf16x8_t *>(
                    rows_lds + row * RW + 4 * ((2 * ks + (lane >> 5)) ^ (row & (CH - 1))));
            }
        };

        const int wk = wave / WQ, wq = wave % WQ;   // wave: BT/KW keys x BQ/WQ queries
        const int lr = lane & 31, lh = lane >> 5;

        // the query rows pass through the key rows' space; BT >= BQ
        load_rows(qr);
        if constexpr (GATHER) {
            for (int t = tid; t < D + 16; t += NT) dims[t] = static_cast<uint16_t>((t < k ? I[t] : D) * 2);
            for (int r = tid; r < BT; r += NT) rows_lds[r * RW + D / 2] = 0u;    // what padding positions read
        } else {
            if (tid < D / 8) reinterpret_cast<uint4 *>(dims)[tid] = make_uint4(0, 0, 0, 0);
            __syncthreads();
            if (tid < k) dims[I[tid]] = 0xffffu;
            __syncthreads();
            km = reinterpret_cast<const uint4 *>(dims)[tid % CH];
        }
        store_rows();
        __syncthreads();
        bf16x8_t qf[FJ][KSMAX];
#pragma unroll
        for (int j = 0; j < FJ; ++j)
#pragma unroll
            for (int ks = 0; ks < KSMAX; ++ks)
                if (!GATHER || ks < KS) qf[j][ks] = frag((wq * FJ + j) * 32 + lr, ks);
        // Each block walks its key tiles starting at a tile of its own and
        // wrapping around, so that at any moment the blocks store to
        // different column ranges of their rows (all starting at column 0
        // measured about 1.5x slower without the causal mask: the row pieces
        // of simultaneous tiles then share too few memory channels).
        const int rot = (bh * 5 + qt) % nc;
        auto tile_at = [&](int i) { const int t = i + rot; return t_lo + (t >= nc ? t - nc : t); };
        load_rows(key_rsrc(tile_at(0)));
        __syncthreads();
        store_rows();
        __syncthreads();

        // RAG: the last 64 columns of a tile, kept for the next tile's first lines
        constexpr int CC = BQ * 8 / NT;
        uint4 carry[CC];
#pragma unroll
        for (int i = 0; i < CC; ++i) carry[i] = make_uint4(0, 0, 0, 0);
        const bool row8 = Lk % 8 == 0 && (s_mis & 7) == 0;      // every row 16-byte aligned
        for (int it = 0; it < nc; ++it) {
            const int kt = tile_at(it);
            if (it + 1 < nc) load_rows(key_rsrc(tile_at(it + 1)));
            f32x16_t acc[FI][FJ];
#pragma unroll
            for (int i = 0; i < FI; ++i)
#pragma unroll
                for (int j = 0; j < FJ; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KSMAX; ++ks) {
                if (GATHER && ks >= KS) continue;
#pragma unroll
                for (int i = 0; i < FI; ++i) {
                    const bf16x8_t kf = frag((wk * FI + i) * 32 + lr, ks);
#pragma unroll
                    for (int j = 0; j < FJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[j][ks], acc[i][j], 0, 0, 0);
                }
            }
            // acc[i][j][4*gq + r]: key (wk*FI + i)*32 + 8*gq + 4*lh + r, query (wq*FJ + j)*32 + lr
            // a tile whose last key is at most its first query + off has no masked entry
            const bool tile_open = !causal || kt * BT + BT - 1 <= q0 + off;
#pragma unroll
            for (int i = 0; i < FI; ++i)
#pragma unroll
                for (int j = 0; j < FJ; ++j) {
                    const int ql = (wq * FJ + j) * 32 + lr;
                    const int qg = q0 + ql;
#pragma unroll
                    for (int gq = 0; gq < 4; ++gq) {
                        const int kl = (wk * FI + i) * 32 + 8 * gq + 4 * lh;
                        uint32_t w0 = pack_bf16x2(acc[i][j][4 * gq] * scale, acc[i][j][4 * gq + 1] * scale);
                        uint32_t w1 = pack_bf16x2(acc[i][j][4 * gq + 2] * scale, acc[i][j][4 * gq + 3] * scale);
                        if (!tile_open) {
                            const int lim = qg + off - (kt * BT + kl);   // keys kl + r kept iff r <= lim
                            if (lim < 0) w0 = (w0 & 0xffff0000u) | kBf16NegInf;
                            if (lim < 1) w0 = (w0 & 0x0000ffffu) | (static_cast<uint32_t>(kBf16NegInf) << 16);
                            if (lim < 2) w1 = (w1 & 0xffff0000u) | kBf16NegInf;
                            if (lim < 3) w1 = (w1 & 0x0000ffffu) | (static_cast<uint32_t>(kBf16NegInf) << 16);
                        }
                        *reinterpret_cast<uint2 *>(&out_lds[ql * OS + PRE + kl]) = make_uint2(w0, w1);
                    }
                }
            if constexpr (RAG) {
#pragma unroll
                for (int i = 0; i < CC; ++i) {
                    const int v = tid + NT * i;
                    *reinterpret_cast<uint4 *>(&out_lds[(v >> 3) * OS + 8 * (v & 7)]) = carry[i];
                }
            }
            lds_barrier();
            auto lds_chunk = [&](int r, int e) { return *reinterpret_cast<const uint4 *>(&out_lds[r * OS + e]); };
            auto put1 = [&](uint16_t x, int r, int col, bool on) __attribute__((always_inline)) {
                __builtin_amdgcn_raw_buffer_store_b16(x, sr, on ? static_cast<uint32_t>((r * Lk + col) * 2) : 0x80000000u, 0, kStoreAux);
            };
            const int t0 = kt * BT;
            uint4 staged[SR];
            if constexpr (!RAG) {
#pragma unroll
                for (int i = 0; i < SR; ++i) {
                    const int r = row_of(i), col = t0 + 8 * c16;
                    staged[i] = lds_chunk(r, 8 * c16);
                    // unconditional (a column past Lk goes out of range): a branch
                    // here would make the compiler's wait for the next K rows also
                    // wait for these stores
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{staged[i].x, staged[i].y, staged[i].z, staged[i].w}, sr,
                        (ANY ? col + 8 <= Lk : col < Lk) ? static_cast<uint32_t>((r * Lk + col) * 2) : 0x80000000u, 0, kStoreAux);
                }
                if constexpr (ANY) {
                    if (t0 + BT > Lk) {                   // the elements after the row's last whole chunk
#pragma unroll
                        for (int r0 = 0; r0 < BQ; r0 += NT / 8) {
                            const int r = r0 + (tid >> 3), cl = ((Lk - t0) & ~7) + (tid & 7);
                            put1(out_lds[r * OS + cl], r, t0 + cl, t0 + cl < Lk);
                        }
                    }
                }
            } else {
                // whole 128-byte lines: columns t0 - m .. t0 + BT - m - 1 of a row m
                // elements past a line boundary, the first m from the tile before
                const bool first = it == 0 || kt == t_lo, last = it == nc - 1 || kt == t_lo + nc - 1;
                auto put = [&](int i0, auto SHv) __attribute__((always_inline)) {
                    constexpr int SH = decltype(SHv)::value;      // m % 8
#pragma unroll
                    for (int ii = 0; ii < IPR; ++ii) {
                        const int r = row_of(i0 + ii), m = mis(r), e = PRE - (m & ~7) + 8 * c16;
                        uint4 x = lds_chunk(r, e);
                        if constexpr (SH > 0) {
                            // the previous chunk's last SH elements, then this one's first 8 - SH
                            const uint4 p = lds_chunk(r, e - 8);
                            const uint32_t d[8] = {p.x, p.y, p.z, p.w, x.x, x.y, x.z, x.w};
                            constexpr int ds = (8 - SH) >> 1;
                            uint32_t o[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                o[q] = SH & 1 ? __builtin_amdgcn_alignbit(d[ds + q + 1], d[ds + q], 16) : d[ds + q];
                            x = make_uint4(o[0], o[1], o[2], o[3]);
                        }
                        const int col = t0 - m + 8 * c16;
                        __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{x.x, x.y, x.z, x.w}, sr,
                            col + 8 <= Lk && !(first && col < t0) ? static_cast<uint32_t>((r * Lk + col) * 2) : 0x80000000u, 0, kStoreAux);
                    }
                };
#pragma unroll
                for (int u = 0; u < RES; ++u) {
                    switch (mis(wave_u + NWV * u) & 7) {
                    case 0: put(u * IPR, std::integral_constant<int, 0>{}); break;
                    case 1: put(u * IPR, std::integral_constant<int, 1>{}); break;
                    case 2: put(u * IPR, std::integral_constant<int, 2>{}); break;
                    case 3: put(u * IPR, std::integral_constant<int, 3>{}); break;
                    case 4: put(u * IPR, std::integral_constant<int, 4>{}); break;
                    case 5: put(u * IPR, std::integral_constant<int, 5>{}); break;
                    case 6: put(u * IPR, std::integral_constant<int, 6>{}); break;
                    default: put(u * IPR, std::integral_constant<int, 7>{}); break;
                    }
                }
                if (first) {                              // the elements before the first whole chunk
#pragma unroll
                    for (int r0 = 0; r0 < BQ; r0 += NT / 8) {
                        const int r = r0 + (tid >> 3), e = tid & 7, sh = mis(r) & 7;
                        put1(out_lds[r * OS + PRE + e], r, t0 + e, sh > 0 && e < 8 - sh && t0 + e < Lk);
                    }
                }
                if (t0 + BT > Lk) {                       // the elements after the row's last whole chunk
#pragma unroll
                    for (int r0 = 0; r0 < BQ; r0 += NT / 8) {
                        const int r = r0 + (tid >> 3), m = mis(r);
                        const int cl = min((Lk - t0 + m) & ~7, BT) - m + (tid & 7);   // column within the tile
                        put1(out_lds[r * OS + PRE + cl], r, t0 + cl, t0 + cl < Lk && cl < BT - m && !(first && cl < 0));
                    }
                }
                if (last) {
                    // what the next tile's lines would take: m elements per row
                    if (row8) {
#pragma unroll
                        for (int r0 = 0; r0 < BQ; r0 += NT / 8) {
                            const int r = r0 + (tid >> 3), m = mis(r), cl = BT - m + 8 * (tid & 7);
                            const uint4 x = lds_chunk(r, PRE + min(cl, BT - 8));
                            __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{x.x, x.y, x.z, x.w}, sr,
                                cl < BT && t0 + cl < Lk ? static_cast<uint32_t>((r * Lk + t0 + cl) * 2) : 0x80000000u, 0, kStoreAux);
                        }
                    } else {
                        for (int r = wave; r < BQ; r += NWV) {
                            const int cl = BT - mis(r) + lane;
                            put1(out_lds[r * OS + PRE + min(cl, BT - 1)], r, t0 + cl, cl < BT && t0 + cl < Lk);
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < CC; ++i) {
                    const int v = tid + NT * i;
                    carry[i] = lds_chunk(v >> 3, PRE + BT - 64 + 8 * (v & 7));
                }
            }
            if constexpr (ST) {
                // After the stores are issued, so that this work overlaps their
                // drain, and without branches, for the same reason as above.
                // Masked keys hold -inf already; a chunk past Lk is not scores.
#pragma unroll
                for (int i = 0; i < SR; ++i) {
                    const int col = t0 + 8 * c16;
                    const uint32_t w[4] = {staged[i].x, staged[i].y, staged[i].z, staged[i].w};
                    float e[8];
                    float cm = -__builtin_inff();
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        e[2 * q] = col < Lk ? __uint_as_float(w[q] << 16) : -__builtin_inff();
                        e[2 * q + 1] = col < Lk ? __uint_as_float(w[q] & 0xffff0000u) : -__builtin_inff();
                        cm = fmaxf(cm, fmaxf(e[2 * q], e[2 * q + 1]));
                    }
                    const float mm = fmaxf(st_m[i], cm);
                    // with nothing kept so far every term below is exp(-inf) = 0
                    const float mref = mm == -__builtin_inff() ? 0.f : mm;
                    float l = st_l[i] * __expf(st_m[i] - mref);
#pragma unroll
                    for (int q = 0; q < 8; ++q) l += __expf(e[q] - mref);
                    st_m[i] = mm;
                    st_l[i] = l;
                }
            }
            if (it + 1 < nc) store_rows();
            lds_barrier();
        }
    }
    if constexpr (ST) {
#pragma unroll
        for (int i = 0; i < SR; ++i) {
#pragma unroll
            for (int sh = 1; sh < CPR; sh <<= 1) {
                const float m2 = __shfl_xor(st_m[i], sh), l2 = __shfl_xor(st_l[i], sh);
                const float mm = fmaxf(st_m[i], m2);
                if (mm != -__builtin_inff()) {
                    const float a = st_m[i] == -__builtin_inff() ? 0.f : st_l[i] * __expf(st_m[i] - mm);
                    const float c = m2 == -__builtin_inff() ? 0.f : l2 * __expf(m2 - mm);
                    st_m[i] = mm;
                    st_l[i] = a + c;
                }
            }
            const int r = row_of(i);
            if (c16 == 0 && q0 + r < Lq) {
                const int64_t row = static_cast<int64_t>(bh) * Lq + q0 + r;
                const bool empty = !(st_l[i] > 0.f);
                rmax[row] = empty ? 0.f : st_m[i];
                rinv[row] = empty ? 0.f : 1.0f / st_l[i];
            }
        }
    }
    // key tiles wholly above the diagonal: one contiguous run per row, each
    // wave writing whole rows with 1 KiB per store instruction
    const uint32_t ninf2 = 0xff80ff80u;
    const int c0 = max(t_lo, n_compute) * BT, c_end = min(Lk, t_hi * BT);
    for (int r = wave; r < BQ && c0 < c_end; r += NT / 64) {
        // 16-byte vectors from the row's first aligned element on, lanes placed in
        // 128-byte lines as above, and the elements before and after them
        const int row0 = r * Lk, m = (s_mis + row0 + c0) & 63;
        const int head = RAG ? max(0, min((8 - (m & 7)) & 7, c_end - c0)) : 0;
        const int c1 = c0 + head, nv = (c_end - c1) / 8;
        for (int v = lane - (RAG ? ((m + head) & 63) >> 3 : 0); v < nv; v += 64)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{ninf2, ninf2, ninf2, ninf2}, sr,
                !RAG || v >= 0 ? static_cast<uint32_t>((row0 + c1 + 8 * v) * 2) : 0x80000000u, 0, kStoreAux);
        if constexpr (ANY) {
            // lanes 0..7: the elements before, 8..15: after
            const int c = lane < 8 ? c0 + lane : c1 + 8 * max(nv, 0) + lane - 8;
            const bool on = lane < 8 ? lane < head : lane < 16 && c < c_end;
            __builtin_amdgcn_raw_buffer_store_b16(kBf16NegInf, sr,
                on ? static_cast<uint32_t>((row0 + c) * 2) : 0x80000000u, 0, kStoreAux);
        }
    }
}

template <int BM, int BN, int BK>
__global__ __launch_bounds__(256) void qk_f32_kernel(
    const float *__restrict__ Q, const float *__restrict__ Kc, const int32_t *__restrict__ idx,
    float *__restrict__ S, int H, int Hkv, int Lq, int Lk, int D, int k, float scale, int causal) {
    constexpr int TX = 16, TY = 16;
    constexpr int RM = BM / TY, RN = BN / TX;
    __shared__ float As[BK][BM + 1];
    __shared__ float Bs[BK][BN + 1];
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
    const int bh = blockIdx.z, b = bh / H, h = bh % H, g = h / (H / Hkv);
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int off = Lk - Lq;
    const float *Qh = Q + static_cast<int64_t>(bh) * Lq * D;
    const float *Kh = Kc + (static_cast<int64_t>(b) * Hkv + g) * Lk * D;
    const int32_t *I = idx + static_cast<int64_t>(bh) * k;
    float *Sh = S + static_cast<int64_t>(bh) * Lq * Lk;

    float acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) acc[i][j] = 0.f;

    const bool skip = causal && n0 > m0 + BM - 1 + off;
    for (int t0 = 0; t0 < k && !skip; t0 += BK) {
        for (int v = tid; v < BM * BK; v += 256) {
            const int c = v % BK, r = v / BK;
            const int t = t0 + c, m = m0 + r;
            As[c][r] = (t < k && m < Lq) ? Qh[static_cast<int64_t>(m) * D + I[t]] : 0.f;
        }
        for (int v = tid; v < BN * BK; v += 256) {
            const int c = v % BK, r = v / BK;
            const int t = t0 + c, n = n0 + r;
            Bs[c][r] = (t < k && n < Lk) ? Kh[static_cast<int64_t>(n) * D + I[t]] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < BK; ++c) {
            float a[RM], bb[RN];
#pragma unroll
            for (int i = 0; i < RM; ++i) a[i] = As[c][ty + i * TY];
#pragma unroll
            for (int j = 0; j < RN; ++j) bb[j] = Bs[c][tx + j * TX];
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j) acc[i][j] = fmaf(a[i], bb[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            const int m = m0 + ty + i * TY, n = n0 + tx + j * TX;
            if (m < Lq && n < Lk)
                Sh[static_cast<int64_t>(m) * Lk + n] =
                    (causal && n > m + off) ? -__builtin_inff() : acc[i][j] * scale;
        }
}

}  // namespace

bool qk_rows_ok(int64_t Lk, int64_t D, const void *S) {
    // Lk bound: a block's 128 rows of S are addressed with 32-bit byte offsets
    return (D == 64 || D == 128) && Lk % 8 == 0 && Lk <= (1 << 22) &&
           reinterpret_cast<uintptr_t>(S) % 16 == 0;
}

namespace {
// rows of S on 128-byte lines
bool qk_lines(int64_t Lk, const void *S) { return Lk % 64 == 0 && reinterpret_cast<uintptr_t>(S) % 128 == 0; }
// Gathered dims (half the matrix work) where the masked product in 128-key tiles
// no longer hides behind the stores: 32 heads, k = 64, us masked / gathered: 8192
// keys 845 / 790 to 805, without the mask 850 / 813 (8 heads x 8192: 242 / 202).
// Masked in 256-key tiles the first takes 771 to 790, within the runs' spread.
bool qk_gathered(int64_t base, int64_t Lk, int64_t D, int64_t k, const void *S) {
    return D == 128 && k <= 64 && Lk >= 6144 && base >= 256 && qk_lines(Lk, S);
}
}  // namespace

hipError_t launch_qk_rowstats_bf16(const uint16_t *Q, const uint16_t *Kc, const int32_t *idx,
                                   int64_t batch, int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk,
                                   int64_t D, int64_t k, float scale, bool causal, uint16_t *S,
                                   float *rmax, float *rinv, hipStream_t stream) {
    if (!qk_rows_ok(Lk, D, S)) return hipErrorNotSupported;
    const int64_t qb = (Lq + rowk::BQ - 1) / rowk::BQ;
    dim3 grid(static_cast<unsigned>(qb), static_cast<unsigned>(batch * H));
    // A block owns its rows' statistics: one share of the keys.  Two blocks of
    // 128-key tiles per CU where there are blocks for it and for the shortest rows;
    // else 256-key tiles, with gathered dims where few are kept (us at D = 128, 128-key /
    // 256-key / gathered tiles: 4 x 28 heads x 384, k = 103 20 / 31; 1 x 32 x 2048, k = 64
    // 80 / 90 / 90; 1 x 32 x 3776, k = 103 229 / 271; 1 x 8 x 3072, k = 32 74 / 60 / 55).
    const int64_t base = qb * batch * H;
    const bool narrow = D == 64 || Lk <= 400 || (base > 256 && Lk < 4608 && (Lk < 2560 || base >= 800));
    auto kern = D == 64 ? qk_bf16_rows_kernel<64, 1, 256, 128, true>
              : narrow ? qk_bf16_rows_kernel<128, 2, 256, 128, true>
              : k <= 48 || qk_gathered(base, Lk, D, k, S) ? qk_bf16_rows_kernel<128, 1, 512, 256, true, 0, true>
                                                          : qk_bf16_rows_kernel<128, 2, 512, 256, true>;
    hipLaunchKernelGGL(kern, grid, dim3(narrow ? 256 : 512), 0, stream, Q, Kc, idx, S,
                       static_cast<int>(H), static_cast<int>(Hkv), static_cast<int>(Lq),
                       static_cast<int>(Lk), static_cast<int>(k), scale, causal ? 1 : 0, 1, rmax, rinv);
    return hipGetLastError();
}

hipError_t launch_qk_bf16(const uint16_t *Q, const uint16_t *Kc, const int32_t *idx,
                          int64_t batch, int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk,
                          int64_t D, int64_t k, float scale, bool causal, uint16_t *S,
                          hipStream_t stream) {
    // 32-bit byte offsets into a block's 128 rows of S
    if ((D == 64 || D == 128) && Lk <= (1 << 22)) {
        // Which form (us at D = 128 unless said; the others in brackets).
        const int64_t qb = (Lq + rowk::BQ - 1) / rowk::BQ, base = qb * batch * H;
        const bool lines = qk_lines(Lk, S), rows16 = qk_rows_ok(Lk, D, S);
        const bool square = 2 * Lq > Lk, half = causal && square;   // half: about half the tiles have a product
        const bool shared = H > Hkv;                       // neighbouring blocks read the same keys
        // Long rows that share lines, once S is past the 256 MB that the memory side
        // cache absorbs: pieces shifted to lines, unless every other row starts at half
        // a line.  1 x 28 heads x 2712 keys, k = 64 121 [128-key tiles 159, gathered 154],
        // 1 x 64 x 2001 (odd) 177 [208], 4 x 32 x 1416 163 [206]; at 257 MB, 1 x 64 x 1416
        // 80 [gathered 72]; 1 x 28 x 4000 (half lines) 252 [gathered 243].
        const bool past = !lines && Lk >= 1408 && 2 * batch * H * Lq * Lk >= 320000000;
        const bool shift = past && (D == 64 || !(Lk % 32 == 0 && reinterpret_cast<uintptr_t>(S) % 64 == 0));
        // Gathered dims (half the matrix work at k = 64), with 256-key tiles, one block
        // per CU: for the longest rows and the half-line ones above; causal from 3968 keys
        // on (1 x 32 heads x 4096, k = 32: 218 [237]); without the mask from 1280 keys on
        // if few dims are kept or rows share lines (1 x 64 x 4096, k = 32: 386 [436]; 1 x 8 x
        // 3584 40 [43]; k = 64: 445 [447]).  Rows on lines whose heads share no keys: not,
        // or later (32 / 32 heads x 4096, k = 64 248 [240], x 5504 437 [469]; 16 / 16 x 3072,
        // k = 32, no mask 96 [74]).
        const bool gathered = D == 128 && k <= 64 && rows16 && !shift &&
            (qk_gathered(base, Lk, D, k, S) || past ||
             (half ? (base >= 512 && Lk >= (shared || !lines ? 3968 : 4608)) || (k <= 48 && base >= 1024 && Lk >= 1000 && Lk < 1280)
                   : square && (!lines || (shared && k <= 48)) && ((base >= 512 && Lk >= 1280) || (base >= 160 && Lk >= 2000))));
        // 256-key tiles (512-byte row pieces) otherwise for the longest rows (8192 keys,
        // k = 128: 760 to 788 [838]) and wherever S is past the cache off the lines
        const bool wide = D == 128 && (gathered || past || (lines && Lk >= 6144 && base >= 256));
        const int64_t tiles = (Lk + (wide ? 255 : 127)) / (wide ? 256 : 128);
        // Shares of the keys, two blocks of 128-key tiles per CU.  Causal rows of middle
        // length: three, which start and end at different times (1 x 64 x 1536, k = 64 66
        // [1: 77, 2: 76], 4 x 32 x 2240 258 [284, 301], 1 x 16 x 3000 77 [99, 90], 64 dims 1 x
        // 28 x 1411 25 [33, 30]; at 4096 keys 242 [244, 238]).  Otherwise, below 160 blocks,
        // as many as give 512; up to there the count with the fewest tiles in all rounds (1 x
        // 28 heads x 1000 keys, 224 blocks: 2 shares 15.6 [1: 20.0, 3: 19.0]; 4 x 32 x 384, 384
        // blocks: 1 share 13.2 [2: 17.8]), two rather than one where that costs little (1 x
        // 16 x 2240, 288 blocks: 42 [52]).  Long rows on lines: two (4096 keys, k = 128, no
        // mask; heads that share no keys from 1024 on, 64 / 64 x 1280 60 [73], 32 / 32 x 4096
        // 227 [320]).
        const bool three = half && Lk >= 1280 && Lk < 3968 &&
            (base > 512 || (base == 512 && !shared) || (base < 512 && base >= 171 && (base <= 200 || base >= 270) && tiles >= (D == 64 ? 11 : 20)));
        int64_t C = 1;
        if (wide || shift) {
            C = 1;
        } else if (three) {
            C = 3;
        } else if (base < 160) {
            C = (512 + base - 1) / base;
        } else if (base < 512) {
            int64_t least = tiles;
            const bool two = base <= 352 || !shared || (tiles >= 18 && base <= 448);
            for (int64_t c = 2; c <= (512 + base - 1) / base; ++c) {
                const int64_t t = (base * c + 511) / 512 * ((tiles + c - 1) / c);
                if (t < least || (c == 2 && two && t <= least + (tiles >= 9))) { least = t; C = c; }
            }
        } else if (lines && (shared ? base > 512 && Lk >= 2048 && (D == 128 || half || Lk < 4096)
                                    : square && Lk >= 1024)) {
            C = 2;
        }
        if (C > tiles) C = tiles;
        const int64_t tpc = (tiles + C - 1) / C;
        C = (tiles + tpc - 1) / tpc;                      // no empty share
        const dim3 grid(static_cast<unsigned>(qb * C), static_cast<unsigned>(batch * H));
        auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, dim3(wide ? 512 : 256), 0, stream, Q, Kc, idx, S,
                               static_cast<int>(H), static_cast<int>(Hkv), static_cast<int>(Lq),
                               static_cast<int>(Lk), static_cast<int>(k), scale, causal ? 1 : 0,
                               static_cast<int>(C), nullptr, nullptr);
            return hipGetLastError();
        };
        if (gathered) return run(qk_bf16_rows_kernel<128, 1, 512, 256, false, 0, true>);
        if (shift) return wide ? run(qk_bf16_rows_kernel<128, 2, 512, 256, false, 2>) : run(qk_bf16_rows_kernel<64, 1, 256, 128, false, 2>);
        if (wide) return run(qk_bf16_rows_kernel<128, 2, 512, 256>);
        if (rows16) return D == 64 ? run(qk_bf16_rows_kernel<64, 1, 256, 128>) : run(qk_bf16_rows_kernel<128, 2, 256, 128>);
        return D == 64 ? run(qk_bf16_rows_kernel<64, 1, 256, 128, false, 1>) : run(qk_bf16_rows_kernel<128, 2, 256, 128, false, 1>);
    }
    constexpr int BM = 128, BN = 128, BK = 32, WM = 2, WN = 2;
    dim3 grid(static_cast<unsigned>((Lk + BN - 1) / BN), static_cast<unsigned>((Lq + BM - 1) / BM),
              static_cast<unsigned>(batch * H));
    hipLaunchKernelGGL((qk_bf16_kernel<BM, BN, BK, WM, WN>), grid, dim3(WM * WN * kWave), 0, stream,
                       Q, Kc, idx, S, static_cast<int>(H), static_cast<int>(Hkv),
                       static_cast<int>(Lq), static_cast<int>(Lk), static_cast<int>(D),
                       static_cast<int>(k), scale, causal ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_qk_f32(const float *Q, const float *Kc, const int32_t *idx, int64_t batch,
                         int64_t H, int64_t Hkv, int64_t Lq, int64_t Lk, int64_t D, int64_t k,
                         float scale, bool causal, float *S, hipStream_t stream) {
    constexpr int BM = 64, BN = 64, BK = 16;
    dim3 grid(static_cast<unsigned>((Lk + BN - 1) / BN), static_cast<unsigned>((Lq + BM - 1) / BM),
              static_cast<unsigned>(batch * H));
    hipLaunchKernelGGL((qk_f32_kernel<BM, BN, BK>), grid, dim3(256), 0, stream, Q, Kc, idx, S,
                       static_cast<int>(H), static_cast<int>(Hkv), static_cast<int>(Lq),
                       static_cast<int>(Lk), static_cast<int>(D), static_cast<int>(k), scale,
                       causal ? 1 : 0);
    return hipGetLastError();
}

}  // namespace rmm
