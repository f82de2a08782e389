// TopK over each unit's energies (Sec. 3.2: I = TopK({s_j}, ceil(rho d))),
// returned as an ascending index list.
//
// One workgroup per selection unit.  Each float64 energy is mapped to a
// 64-bit key whose unsigned order is the order of the values (NaN above
// +inf, -0 == +0), so the whole selection is integer work: an MSB-first
// radix select with 8-bit digits narrows the keys down to the bucket holding
// the k-th largest, using LDS histograms with integer atomics
// (order-independent counts).  It starts below the leading bits every key
// shares and stops as soon as that bucket is taken whole or holds at most
// kRankMax keys (kRankShort in short units); those are then ranked directly (a
// wave per key: ballots over the others).  Keys tied with the k-th key are taken lowest index first, and
// the kept indices are compacted in ascending order with one workgroup prefix
// scan.  Each thread owns a contiguous chunk of keys, kept in registers when it
// fits.  Units of up to 128 keys (attention heads) skip the radix passes: every
// thread ranks its own key against all of them.  For a unit of one token (a
// decode step) the keys come straight from the token's activations: 16 (bf16)
// or 31 (fp32) key bits, so at most two passes for bf16 and four for fp32.
//
// What bounds it is the chain of dependent LDS passes and barriers of one
// workgroup.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rmm {

namespace {

__device__ __forceinline__ uint64_t order_key(double d) {
    uint64_t u = __double_as_longlong(d);
    if (d != d) u = 0x7ff8000000000000ull;          // every NaN -> one quiet NaN
    if (u == 0x8000000000000000ull) u = 0;          // -0 ties with +0
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Inclusive prefix sum over the wave: shifts within rows of 16 lanes, then
// the last lane of a row into the next one(s) (data-parallel moves, no LDS).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto step = [](uint32_t v, auto ctrl, auto rows) {
        return v + static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
                       0, static_cast<int>(v), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
    };
    using all = std::integral_constant<int, 0xF>;
    x = step(x, std::integral_constant<int, 0x111>{}, all{});
    x = step(x, std::integral_constant<int, 0x112>{}, all{});
    x = step(x, std::integral_constant<int, 0x114>{}, all{});
    x = step(x, std::integral_constant<int, 0x118>{}, all{});
    x = step(x, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});
    x = step(x, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});
#endif
    return x;
}

// Exclusive prefix sum of v over the workgroup in thread order (one barrier;
// `buf`, one word per wave, may be reused only after another).
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *buf) {
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t incl = wave_inclusive_scan(v);
    if (lane == kWave - 1) buf[w] = incl;
    __syncthreads();
    const uint32_t x = wave_inclusive_scan(lane < NW ? buf[lane] : 0u);
    const uint32_t before = w == 0 ? 0u : static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), w > 0 ? w - 1 : 0));
    return before + incl - v;
}

// Sum of the wave-uniform v over the waves before this one (one barrier).
template <int NT>
__device__ __forceinline__ uint32_t waves_before(uint32_t v, uint32_t *buf) {
    const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (lane == 0) buf[w] = v;
    __syncthreads();
    uint32_t r = 0;
#pragma unroll
    for (int q = 0; q < NT / kWave; ++q) r += q < w ? buf[q] : 0u;
    return r;
}

// The 256-bin histogram in HR copies (lane % HR counts into one of them, HS
// words apart so that one digit's copies sit in different banks): threads
// 0..255 add up bin 255 - tid, clear its copies for the next pass and find
// the bin where the descending running count reaches `need`.  Called by the
// whole workgroup after the counting; out[0..2] = digit, keys above it, its
// size, valid after the barrier this ends with.
constexpr int HR = 16, HS = 257;
__device__ __forceinline__ void pick_digit(uint32_t *hcopy, uint32_t need, uint32_t *wtot, uint32_t *out) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    uint32_t h = 0, incl = 0;
    __syncthreads();
    if (tid < 256) {
#pragma unroll
        for (int r = 0; r < HR; ++r) {
            h += hcopy[r * HS + 255 - tid];
            hcopy[r * HS + 255 - tid] = 0;
        }
        incl = wave_inclusive_scan(h);
        if (lane == kWave - 1) wtot[w] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t run = incl - h;
#pragma unroll
        for (int q = 0; q < 3; ++q) run += q < w ? wtot[q] : 0u;
        if (run < need && need <= run + h) {
            out[0] = 255 - tid;
            out[1] = run;
            out[2] = h;
        }
    }
    __syncthreads();
}

// Where the keys come from: a unit's float64 energies, or (a unit of one
// token) the token's bf16 or fp32 activations.  For one token the energy of
// index j is x_j^2, which is exact in float64 and orders like |x_j|, whose
// IEEE bits (sign cleared) are already an unsigned order key: equal |x| tie
// exactly as equal squares do, +inf ranks above every finite value and every
// NaN is mapped to one key above +inf -- the order of the energy keys.
enum KeySrc { kEnergy = 0, kTokenBf16 = 1, kTokenF32 = 2 };

template <int SRC>
__device__ __forceinline__ uint64_t load_key(const void *row, int64_t j) {
    if constexpr (SRC == kEnergy) {
        return order_key(static_cast<const double *>(row)[j]);
    } else if constexpr (SRC == kTokenBf16) {
        uint32_t a = static_cast<const uint16_t *>(row)[j] & 0x7fffu;
        return a > 0x7f80u ? 0x7fc0u : a;
    } else {
        uint32_t a = static_cast<const uint32_t *>(row)[j] & 0x7fffffffu;
        return a > 0x7f800000u ? 0x7fc00000u : a;
    }
}

// Units of K <= NT / 4 keys: the quad of lanes t ranks key t against all of
// them (each lane a quarter; ties to the lower index) and keeps it if fewer
// than k come before it.  128 keys, us against the radix passes: 32 units 4.8 /
// 5.8, 1024 units 6.2 / 8.2.
template <int NT, int SRC>
__global__ __launch_bounds__(NT) void select_rank_kernel(const void *__restrict__ src, int64_t ld, int K,
                                                         int k, int32_t *__restrict__ idx) {
    constexpr int KP = NT / 4;
    __shared__ __attribute__((aligned(16))) uint64_t keys[KP];
    __shared__ uint32_t wcnt[NT / kWave];
    constexpr int esize = SRC == kEnergy ? 8 : SRC == kTokenBf16 ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int t = tid >> 2, part = tid & 3;
    const void *e = static_cast<const char *>(src) + static_cast<int64_t>(blockIdx.x) * ld * esize;
    int32_t *out = idx + static_cast<int64_t>(blockIdx.x) * k;
    if (k == K) {                       // everything is kept (512 units of 152: 2.3 us; 8.1 when ranked)
        if (tid < K) out[tid] = tid;
        return;
    }
    if (tid < KP) keys[tid] = tid < K ? load_key<SRC>(e, tid) : 0ull;
    __syncthreads();
    const uint64_t u = keys[t];
    int before = 0;
#pragma unroll 8
    for (int j = part; j < KP; j += 4) {         // keys past K are 0 and come after every real one
        const uint64_t o = keys[j];
        before += o > u || (o == u && j < t);
    }
#if defined(__HIP_DEVICE_COMPILE__)
    before += __builtin_amdgcn_update_dpp(0, before, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    before += __builtin_amdgcn_update_dpp(0, before, 0x4E, 0xF, 0xF, false);   // lane ^ 2
#endif
    const bool keep = part == 0 && t < K && before < k;
    const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
    if (lane == 0) wcnt[w] = static_cast<uint32_t>(__builtin_popcountll(m));
    __syncthreads();
    uint32_t pos = static_cast<uint32_t>(__builtin_popcountll(m & ((1ull << lane) - 1)));
#pragma unroll
    for (int q = 0; q < NT / kWave; ++q) pos += q < w ? wcnt[q] : 0u;
    if (keep) out[pos] = t;
}

// NT threads; C keys per thread held in registers (REG) or re-read from
// memory (REG == false, `cpt` per thread at run time).  A wave owns a
// contiguous run of the keys, its lanes every 64th of it (whole-line loads
// and stores; positions come from ballots).  Unit u's keys start at element
// u * ld of `src`.  Measured (random energies with 1 % outliers, k = K / 2):
// 10.8 -> 7.0 us at K = 4096 and 24.9 -> 15.2 at K = 14336, against radix
// passes down to the last digit over keys owned in runs per thread.
constexpr int kRankMax = 128;      // ranked at once: two per lane (256: 9.6 us instead of 6.4 at K = 1024)
// Of up to 1024 keys a radix pass costs less than ranking more than a few (us for
// 257 keys with a limit of 128 / 24: 256 units 7.4 / 6.1, 4096 units 32.3 / 26.2;
// from 800 keys on limits of 16 to 128 differ by less than 2 %).
constexpr int kRankShort = 32;
template <int NT, int C, bool REG, int SRC>
__global__ __launch_bounds__(NT) void select_kernel(const void *__restrict__ src, int64_t ld,
                                                    int64_t K, int64_t k, int cpt,
                                                    int32_t *__restrict__ idx) {
    constexpr int NW = NT / kWave;
    __shared__ uint32_t hcopy[HR * HS];
    __shared__ uint32_t scan_buf[NW], wtot[4], s_pick[3], s_n;
    __shared__ uint32_t s_min[NW], s_max[NW];
    __shared__ uint64_t cand_key[kRankMax], s_thr;
    __shared__ int32_t cand_idx[kRankMax], s_tie;

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    constexpr int esize = SRC == kEnergy ? 8 : SRC == kTokenBf16 ? 2 : 4;
    const void *e = static_cast<const char *>(src) + static_cast<int64_t>(blockIdx.x) * ld * esize;
    int32_t *out = idx + static_cast<int64_t>(blockIdx.x) * k;
    const int chunk = REG ? C : cpt;
    // key c of this lane is index c0 + 64 * c
    const int64_t c0 = static_cast<int64_t>(wave) * chunk * kWave + lane;
    const uint64_t below = (1ull << lane) - 1;

    if (k == K) {                       // everything is kept
        for (int64_t j = tid; j < K; j += NT) out[j] = static_cast<int32_t>(j);
        return;
    }

    uint64_t keys[REG ? C : 1];
    if constexpr (REG) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int64_t j = c0 + kWave * c;
            keys[c] = j < K ? load_key<SRC>(e, j) : 0ull;
        }
    }
    for (int i = tid; i < HR * HS; i += NT) hcopy[i] = 0;
    if (tid == 0) s_n = 0;
    auto key_at = [&](int c) -> uint64_t {
        if constexpr (REG) return keys[c];
        else return load_key<SRC>(e, c0 + static_cast<int64_t>(kWave) * c);
    };
    const int n_own = static_cast<int>(max<int64_t>(0, min<int64_t>(chunk, (K - c0 + kWave - 1) / kWave)));
    // f over the lane's places (each) or the keys it has (own); unrolled where they
    // are held (indexed at run time they would live in scratch)
    auto each = [&](auto &&f) {
        if constexpr (REG) {
#pragma unroll
            for (int c = 0; c < C; ++c) f(c);
        } else {
            for (int c = 0; c < chunk; ++c) f(c);
        }
    };
    auto own = [&](auto &&f) {
        if constexpr (REG) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (c < n_own) f(c);
        } else {
            for (int c = 0; c < n_own; ++c) f(c);
        }
    };

    // The leading bits shared by every key need no pass (energies of one
    // unit usually share sign and most of the exponent): take the workgroup's
    // smallest and largest high word (a token's keys have only a low word)
    // and start below their common prefix, so the first pass already spreads
    // the keys over its buckets.
    constexpr int SH = SRC == kEnergy ? 32 : 0;
    uint32_t kmin = ~0u, kmax = 0;
    own([&](int c) {
        const uint32_t u = static_cast<uint32_t>(key_at(c) >> SH);
        kmin = min(kmin, u);
        kmax = max(kmax, u);
    });
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        kmin = min(kmin, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmin), o, kWave)));
        kmax = max(kmax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmax), o, kWave)));
    }
    if (lane == 0) { s_min[wave] = kmin; s_max[wave] = kmax; }
    __syncthreads();
    kmin = s_min[0];
    kmax = s_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        kmin = min(kmin, s_min[w]);
        kmax = max(kmax, s_max[w]);
    }
    // top: the highest bit not yet fixed
    int top = kmin == kmax ? SH - 1 : SH + 31 - __builtin_clz(kmin ^ kmax);
    uint64_t mask = top == 63 ? 0ull : (~0ull << (top + 1));
    uint64_t prefix = (static_cast<uint64_t>(kmax) << SH) & mask;
    uint32_t need = static_cast<uint32_t>(k);
    uint32_t *hmine = hcopy + (tid % HR) * HS;
    // keys above `prefix` (under `mask`) are kept, and keys equal to it up to index `tie`
    int64_t tie = -1;
    bool decided = false;
    while (top >= 0) {
        // digit: bits top .. shift (up to 8 of them)
        const int shift = max(0, top - 7);
        const uint64_t dmask = (1ull << (top - shift + 1)) - 1;
        own([&](int c) {
            const uint64_t u = key_at(c);
            if ((u & mask) == prefix) atomicAdd(&hmine[(u >> shift) & dmask], 1u);
        });
        pick_digit(hcopy, need, wtot, s_pick);
        need -= s_pick[1];
        prefix |= static_cast<uint64_t>(s_pick[0]) << shift;
        mask |= dmask << shift;
        top = shift - 1;
        const uint32_t n = s_pick[2];
        if (n == need) { tie = K; decided = true; break; }      // the whole bucket is kept
        if (n <= (REG && NT * C <= 1024 ? kRankShort : kRankMax)) {
            // rank the bucket's keys: the one with need - 1 before it is the k-th
            own([&](int c) {
                const uint64_t u = key_at(c);
                if ((u & mask) == prefix) {
                    const uint32_t p = atomicAdd(&s_n, 1u);
                    cand_key[p] = u;
                    cand_idx[p] = static_cast<int32_t>(c0 + kWave * c);
                }
            });
            __syncthreads();
            uint64_t ck[kRankMax / kWave];
            int32_t ci[kRankMax / kWave];
#pragma unroll
            for (int q = 0; q < kRankMax / kWave; ++q) {
                const uint32_t j = static_cast<uint32_t>(lane + kWave * q);
                ck[q] = j < n ? cand_key[j] : 0ull;
                ci[q] = j < n ? cand_idx[j] : 0x7fffffff;     // past the end: before no candidate
            }
            for (uint32_t i = wave; i < n; i += NW) {
                const uint64_t ki = cand_key[i];
                const int32_t ii = cand_idx[i];
                uint32_t before = 0;
#pragma unroll
                for (int q = 0; q < kRankMax / kWave; ++q)
                    before += static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(
                        ck[q] > ki || (ck[q] == ki && ci[q] < ii))));
                if (before == need - 1 && lane == 0) { s_thr = ki; s_tie = ii; }
            }
            __syncthreads();
            prefix = s_thr;
            mask = ~0ull;
            tie = s_tie;
            decided = true;
            break;
        }
    }
    if (!decided) {
        // more than kRankMax equal keys at the threshold: keep the first
        // `need` of them by index
        auto tied = [&](int c) { return c < n_own && (key_at(c) & mask) == prefix; };
        uint32_t n_cand = 0;
        each([&](int c) {
            n_cand += static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(tied(c))));
        });
        uint32_t cand = waves_before<NT>(n_cand, scan_buf);
        each([&](int c) {
            const bool t = tied(c);
            const uint64_t m = __builtin_amdgcn_ballot_w64(t);
            if (t && cand + static_cast<uint32_t>(__builtin_popcountll(m & below)) == need - 1)
                s_tie = static_cast<int32_t>(c0 + static_cast<int64_t>(kWave) * c);
            cand += static_cast<uint32_t>(__builtin_popcountll(m));
        });
        __syncthreads();
        tie = s_tie;
    }

    auto kept = [&](int c) {
        if (c >= n_own) return false;
        const uint64_t p = key_at(c) & mask;
        return p > prefix || (p == prefix && c0 + static_cast<int64_t>(kWave) * c <= tie);
    };
    uint32_t n_sel = 0;
    each([&](int c) {
        n_sel += static_cast<uint32_t>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(kept(c))));
    });
    uint32_t pos = waves_before<NT>(n_sel, scan_buf);
    each([&](int c) {
        const bool keep = kept(c);
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (keep)
            out[pos + static_cast<uint32_t>(__builtin_popcountll(m & below))] =
                static_cast<int32_t>(c0 + static_cast<int64_t>(kWave) * c);
        pos += static_cast<uint32_t>(__builtin_popcountll(m));
    });
}

// One bf16 token per workgroup (a decode step), K <= 32 * 1024 (at most
// 32768 keys, so both 16-bit halves of the packed scan below hold): the keys are
// the 15 magnitude bits, so the k-th largest key is found in at most two
// histogram passes (bits 14..7, then 6..0), each of the NT threads owning C
// consecutive keys loaded as 16-byte vectors.  The kept set is then
// written in ascending order after one scan of a packed pair per thread
// (keys above the threshold | ties with it << 16): a kept key's slot is the
// number of kept keys before it, i.e. keys above before it plus
// min(ties before it, ties kept).
template <int NT, int C>
__device__ __forceinline__ void select_token16(const uint16_t *__restrict__ x, int K, int k,
                                               int32_t *__restrict__ out) {
    static_assert(C % 8 == 0 && C <= 32 && NT >= 256 && NT <= 1024, "chunk");
    // The keys of a token bunch up in a few digits (one per binary exponent),
    // so one histogram would take most of a wave's 64 increments on one
    // word: hence its copies.
    __shared__ uint32_t hcopy[HR * HS];
    __shared__ uint32_t scan_buf[NT / kWave], wtot[4], s_pick[3];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    if (k == K) {                       // everything is kept
        for (int j = tid; j < K; j += NT) out[j] = j;
        return;
    }
    const int c0 = tid * C;
    // keys past K are marked with bit 15 and never counted
    uint32_t key[C];
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x), 0, static_cast<uint32_t>(K) * 2u, 0x00020000);
#pragma unroll
    for (int q = 0; q < C / 8; ++q) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(xr, static_cast<uint32_t>(c0 + 8 * q) * 2u, 0, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t h = (v[e / 2] >> (16 * (e % 2))) & 0x7fffu;
            key[8 * q + e] = c0 + 8 * q + e < K ? (h > 0x7f80u ? 0x7fc0u : h) : 0x8000u;
        }
    }
    for (int j = tid; j < HR * HS; j += NT) hcopy[j] = 0;
    // pass 1 over bits 14..7, pass 2 over bits 6..0 of the keys in the chosen bucket
    int need = k, thr = -1, take_ties = 0;
    int prefix = -1;                    // pass-1 digit, once chosen
    uint32_t *hmine = hcopy + (lane % HR) * HS;
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const uint32_t u = key[c];
            if (u & 0x8000u) continue;
            if (pass == 0) atomicAdd(&hmine[u >> 7], 1u);
            else if (static_cast<int>(u >> 7) == prefix) atomicAdd(&hmine[u & 0x7fu], 1u);
        }
        pick_digit(hcopy, static_cast<uint32_t>(need), wtot, s_pick);
        const int d = static_cast<int>(s_pick[0]), nb = need - static_cast<int>(s_pick[1]);
        const int size = static_cast<int>(s_pick[2]);          // keys of this bucket, nb of them to keep
        if (pass == 0) {
            if (size == nb) { thr = (d << 7) - 1; take_ties = 0; break; }   // the whole bucket
            prefix = d;
            need = nb;
        } else {
            thr = (prefix << 7) | d;    // the k-th largest key; keep nb of its ties
            take_ties = nb;
        }
    }
    // compaction: keys above thr, then the first take_ties keys equal to thr
    uint32_t above = 0, ties = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int u = static_cast<int>(key[c]);
        above += u < 0x8000 && u > thr;
        ties += u == thr;
    }
    const uint32_t pre = block_exclusive_scan<NT>(above | (ties << 16), scan_buf);
    int sa = static_cast<int>(pre & 0xffffu), st = static_cast<int>(pre >> 16);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int u = static_cast<int>(key[c]);
        if (u < 0x8000 && u > thr) {
            out[sa + min(st, take_ties)] = c0 + c;
            ++sa;
        } else if (u == thr) {
            if (st < take_ties) out[sa + st] = c0 + c;
            ++st;
        }
    }
}

template <int NT, int C>
__global__ __launch_bounds__(NT) void select_token16_kernel(const uint16_t *__restrict__ X,
                                                            int64_t ldx, int K, int k,
                                                            int32_t *__restrict__ idx) {
    select_token16<NT, C>(X + static_cast<int64_t>(blockIdx.x) * ldx, K, k,
                          idx + static_cast<int64_t>(blockIdx.x) * k);
}

// the token selection of several groups in one launch: workgroup (b, g)
// takes unit b of group g
__global__ __launch_bounds__(1024) void select_token16_grouped_kernel(GemvGroups G) {
    const GemvGroup &q = G.g[blockIdx.y];
    if (q.K > kToken16MaxK) return;              // selected by a launch of its own
    const uint16_t *x = q.X + static_cast<int64_t>(blockIdx.x) * q.ldx;
    int32_t *out = q.idx_out + static_cast<int64_t>(blockIdx.x) * q.k;
    if (q.K <= 16 * 1024) select_token16<1024, 16>(x, q.K, q.k, out);   // uniform per workgroup
    else select_token16<1024, 32>(x, q.K, q.k, out);
}

template <int NT, int C>
hipError_t launch_token16(const void *X, int64_t ldx, int64_t B, int64_t K, int64_t k, int32_t *idx,
                          hipStream_t stream) {
    hipLaunchKernelGGL((select_token16_kernel<NT, C>), dim3(static_cast<unsigned>(B)), dim3(NT), 0, stream,
                       static_cast<const uint16_t *>(X), ldx, static_cast<int>(K), static_cast<int>(k), idx);
    return hipGetLastError();
}

template <int NT, int C, bool REG, int SRC>
hipError_t launch(const void *src, int64_t ld, int64_t B, int64_t K, int64_t k, int cpt,
                  int32_t *idx, hipStream_t stream) {
    hipLaunchKernelGGL((select_kernel<NT, C, REG, SRC>), dim3(static_cast<unsigned>(B)), dim3(NT), 0,
                       stream, src, ld, K, k, cpt, idx);
    return hipGetLastError();
}

template <int SRC>
hipError_t launch_src(const void *src, int64_t ld, int64_t B, int64_t K, int64_t k, int32_t *idx,
                      hipStream_t stream) {
    if (K <= 128) {
        hipLaunchKernelGGL((select_rank_kernel<512, SRC>), dim3(static_cast<unsigned>(B)), dim3(512), 0, stream, src,
                           ld, static_cast<int>(K), static_cast<int>(k), idx);
        return hipGetLastError();
    }
    // one key per thread (us, radix / every key ranked by 1024 threads: 1 x 160 4.7 / 5.7,
    // 512 x 160 6.7 / 8.9, 4096 x 256 20.5 / 44.9)
    if (K <= 256) return launch<256, 1, true, SRC>(src, ld, B, K, k, 1, idx, stream);
    // Half as many threads with twice the keys where several units share a CU and the
    // fixed work of a workgroup adds up (us at half / all threads: 768 x 512 8.2 / 8.7,
    // 4096 x 512 22.6 / 28.0, 2048 x 800 15.1 / 18.0, 320 x 8192 19.1 / 22.7, 2048 x 8192
    // 73.5 / 96.0; 256 x 512 6.7 / 6.3, 512 x 800 8.3 / 8.1, 256 x 8192 16.2 / 13.9).
    const bool half = B > 256;
    if (K <= 512 && half) return launch<256, 2, true, SRC>(src, ld, B, K, k, 2, idx, stream);
    if (K <= 512) return launch<512, 1, true, SRC>(src, ld, B, K, k, 1, idx, stream);
    if (K <= 1024 && B >= 1024) return launch<256, 4, true, SRC>(src, ld, B, K, k, 4, idx, stream);
    if (K <= 1024) return launch<512, 2, true, SRC>(src, ld, B, K, k, 2, idx, stream);
    if (K <= 2048) return launch<512, 4, true, SRC>(src, ld, B, K, k, 4, idx, stream);
    if (K <= 4096) return launch<1024, 4, true, SRC>(src, ld, B, K, k, 4, idx, stream);
    if (K <= 8192 && half) return launch<512, 16, true, SRC>(src, ld, B, K, k, 16, idx, stream);
    if (K <= 8192) return launch<1024, 8, true, SRC>(src, ld, B, K, k, 8, idx, stream);
    if (K <= 16384) return launch<1024, 16, true, SRC>(src, ld, B, K, k, 16, idx, stream);
    // 32 keys of 64 bits per thread do not all fit its registers (340 bytes of
    // scratch); reading the keys again is faster (us, energies, re-read / held: 1 x
    // 16801 32 / 43, 64 x 16801 33 / 55, 1024 x 16801 155 / 299, 1 x 28672 48 / 47, 512 x
    // 28672 119 / 169; fp32 tokens 256 x 28672 59 / 64) unless they are energies past
    // what the L2s hold and in one round of workgroups (256 x 28672 98 / 71, 128 x
    // 24000 75 / 65; 257 x 28672 98 / 122).  Held and indexed at run time, all of
    // the keys lay in scratch: 50, 66, 373, 57, 192; 73; 79, 71, 138.
    if constexpr (SRC == kEnergy) {
        if (K <= 32768 && B <= 256 && B * K >= 3000000)
            return launch<1024, 32, true, SRC>(src, ld, B, K, k, 32, idx, stream);
    }
    const int cpt = static_cast<int>((K + 1023) / 1024);
    return launch<1024, 1, false, SRC>(src, ld, B, K, k, cpt, idx, stream);
}

// bad[b] = 0 when unit b's list idx[b*k .. b*k+k) is strictly ascending with
// every value in [0, K), else 1 + the first position t that breaks it
// (idx[t] out of range, or idx[t] <= idx[t-1]).  Integer work: the first
// position is an integer minimum over the threads, order-free.
__global__ __launch_bounds__(256) void check_indices_kernel(const int32_t *__restrict__ idx,
                                                            int64_t k, int32_t K,
                                                            int32_t *__restrict__ bad) {
    __shared__ int first;
    const int32_t *I = idx + static_cast<int64_t>(blockIdx.x) * k;
    if (threadIdx.x == 0) first = 0x7fffffff;
    __syncthreads();
    for (int64_t t = threadIdx.x; t < k; t += 256) {
        const int32_t v = I[t];
        if (v < 0 || v >= K || (t > 0 && I[t - 1] >= v)) {
            atomicMin(&first, static_cast<int>(t));      // t grows along a thread's loop
            break;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) bad[blockIdx.x] = first == 0x7fffffff ? 0 : first + 1;
}

}  // namespace

hipError_t launch_check_indices(const int32_t *idx, int64_t B, int64_t k, int64_t K, int32_t *bad,
                                hipStream_t stream) {
    hipLaunchKernelGGL(check_indices_kernel, dim3(static_cast<unsigned>(B)), dim3(256), 0, stream,
                       idx, k, static_cast<int32_t>(K), bad);
    return hipGetLastError();
}

hipError_t launch_select(const double *energy, int64_t B, int64_t K, int64_t k,
                         int32_t *idx, hipStream_t stream) {
    return launch_src<kEnergy>(energy, K, B, K, k, idx, stream);
}

hipError_t launch_select_tokens_grouped(const GemvGroups &G, int64_t B, hipStream_t stream) {
    hipLaunchKernelGGL(select_token16_grouped_kernel, dim3(static_cast<unsigned>(B), static_cast<unsigned>(G.n)),
                       dim3(1024), 0, stream, G);
    hipError_t e = hipGetLastError();
    // groups too wide for the one-pass token kernel: the generic selection
    for (int i = 0; i < G.n && e == hipSuccess; ++i) {
        const GemvGroup &q = G.g[i];
        if (q.K > kToken16MaxK)
            e = launch_select_tokens(q.X, true, B, q.K, q.ldx, q.k, q.idx_out, stream);
    }
    return e;
}

hipError_t launch_select_tokens(const void *X, bool bf16, int64_t B, int64_t K, int64_t ldx,
                                int64_t k, int32_t *idx, hipStream_t stream) {
    // up to 256 channels (a decode step's heads) the generic selection: every key
    // ranked directly, or one key per thread
    if (K > 256 && bf16 && K <= kToken16MaxK && reinterpret_cast<uintptr_t>(X) % 16 == 0 && ldx % 8 == 0) {
        if (K <= 8 * 256) return launch_token16<256, 8>(X, ldx, B, K, k, idx, stream);
        if (K <= 16 * 256) return launch_token16<256, 16>(X, ldx, B, K, k, idx, stream);
        if (K <= 16 * 512) return launch_token16<512, 16>(X, ldx, B, K, k, idx, stream);
        if (K <= 16 * 1024) return launch_token16<1024, 16>(X, ldx, B, K, k, idx, stream);
        return launch_token16<1024, 32>(X, ldx, B, K, k, idx, stream);
    }
    return bf16 ? launch_src<kTokenBf16>(X, ldx, B, K, k, idx, stream)
                : launch_src<kTokenF32>(X, ldx, B, K, k, idx, stream);
}

}  // namespace rmm
