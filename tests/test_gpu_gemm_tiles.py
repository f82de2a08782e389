"""The K-major gathered GEMM's tile choices against the oracle at their edges:
partial tiles in m and n, list tails of a stage and of the list segment held
in LDS, unaligned and very long Y rows, several units."""
import numpy as np
import pytest
import torch

import paper_2608_13426_amd as rmm
import workloads as wl
from tests.gpu_util import gpu, require_gpu, to_device, from_device, check_product

pytestmark = gpu


@pytest.mark.parametrize("B,M,K,N,k,pad", [
    (1, 1, 64, 1, 1, 0),            # 64 x 64 tiles: one row, one column, one index
    (2, 65, 200, 130, 67, 6),       # partial tiles both ways, 8-byte Y rows
    (1, 63, 136, 200, 64, 5),       # odd Y rows: element stores
    (1, 40, 3700, 72, 3584, 0),     # the list is exactly one LDS segment
    (3, 17, 3700, 72, 3585, 0),     # ... and one index more
    (1, 1100, 160, 1040, 97, 0),    # 128 x 128 tiles: staged and partial columns
    (1, 1025, 160, 1023, 160, 4),   # ... odd Y rows
    (2, 700, 3800, 1152, 3700, 4),  # ... two units, two segments, 8-byte Y rows
    (1, 1100, 72, 1139, 40, 1),     # ... 8-byte rows, a last tile of 115 columns
    (2, 1030, 72, 523, 33, 3),      # ... odd columns and rows
    (1, 3000, 72, 3072, 40, 0),     # 256 x 256 tiles (144 of them)
    (1, 130, 72, 128, 33, 1 << 23), # Y rows too long for 32-bit offsets
])
def test_kmajor_tiles(B, M, K, N, k, pad):
    dev = require_gpu()
    xs = wl.random_case(300 + M, (B, M, K), "bf16", n_outlier=2)
    ws = wl.random_case(400 + N, (K, (N + 7) // 8 * 8), "bf16", std=0.02)
    ldxt = (M + 7) // 8 * 8
    xt = np.full((B, K, ldxt), 0x7fc0, np.uint16)          # NaN past M: must reach nothing
    xt[:, :, :M] = xs.transpose(0, 2, 1)
    rng = np.random.default_rng(M + N)
    idx = np.sort(np.stack([rng.choice(K, k, replace=False) for _ in range(B)]), axis=1).astype(np.int32)
    Wd = to_device(ws, "bf16", dev)[:, :N]
    Y = torch.full((B, M, N + pad), 7.0, dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_gemm_kmajor(to_device(xt, "bf16", dev)[:, :, :M], Wd, torch.from_numpy(idx).to(dev), Y[:, :, :N])
    W = wl.decode(ws, "bf16").astype(np.float64)[:, :N]
    got = from_device(Y[:, :, :N])
    for b in range(B):
        X = wl.decode(xs, "bf16")[b].astype(np.float64)
        A = X[:, idx[b]]
        check_product(got[b], A @ W[idx[b]], np.abs(A) @ np.abs(W[idx[b]]), k, "bf16")
    tail = Y[:, :, N:N + 64]
    assert bool((tail == 7.0).all())                       # nothing past N written


@pytest.mark.parametrize("B,M,N,k,pad", [
    (350, 300, 128, 33, 0),         # 1050 blocks of 128 rows: 256 x 128 tiles, partial in m
    (350, 300, 64, 70, 4),          # ... half the columns, 8-byte rows
    (350, 290, 72, 9, 5),           # ... odd rows: element stores
    (520, 257, 5, 64, 0),           # ... one row past a tile, few columns
])
def test_kmajor_tall_tiles(B, M, N, k, pad):
    """Many units of narrow products (value products): partial tiles both ways, guarded columns."""
    dev = require_gpu()
    g = torch.Generator(device=dev).manual_seed(B + N)
    K, ld = 80, (M + 7) // 8 * 8
    xt = torch.full((B, K, ld), float("nan"), dtype=torch.bfloat16, device=dev)    # NaN past M
    xt[:, :, :M] = torch.randn(B, K, M, device=dev, generator=g).bfloat16()
    W = torch.randn(K, (N + 7) // 8 * 8, device=dev, generator=g).bfloat16()
    idx = torch.stack([torch.sort(torch.randperm(K, device=dev, generator=g)[:k]).values for _ in range(B)])
    Y = torch.full((B, M, N + pad), 7.0, dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_gemm_kmajor(xt[:, :, :M], W[:, :N], idx.int().contiguous(), Y[:, :, :N])
    assert bool((Y[:, :, N:] == 7.0).all())
    for b in range(0, B, 7):
        A, Wb = xt[b, idx[b], :M].double().t().cpu().numpy(), W[idx[b], :N].double().cpu().numpy()
        check_product(from_device(Y[b, :, :N]), A @ Wb, np.abs(A) @ np.abs(Wb), k, "bf16")
    for b in range(B):                                     # every unit within a bf16 rounding of a 32-bit product
        ref = xt[b, idx[b], :M].float().t() @ W[idx[b], :N].float()
        assert bool(torch.isfinite(Y[b, :, :N]).all())
        assert float((Y[b, :, :N].float() - ref).abs().max()) <= 2.0 ** -7 * float(ref.abs().max())


@pytest.mark.parametrize("H,Hkv,Lq,Lk,kt", [(2, 1, 1, 40, 33), (4, 2, 129, 129, 60), (2, 2, 300, 420, 200),
                                            (2, 1, 200, 130, 90)])
def test_pv_kmajor_causal_trim(H, Hkv, Lq, Lk, kt):
    """The trimmed K loop: a query tile stops at its last visible token, also
    where Lq != Lk (queries with no visible token get exact zeros)."""
    dev = require_gpu()
    D, ld = 128, (Lq + 7) // 8 * 8
    i, t = np.arange(Lq)[None, :], np.arange(Lk)[:, None]
    p = np.abs(wl.decode(wl.random_case(7, (H, Lk, Lq), "bf16"), "bf16")).astype(np.float32)
    p[:, (t > i + (Lk - Lq))] = 0.0
    pt = np.zeros((1, H, Lk, ld), np.uint16)
    pt[0, :, :, :Lq] = wl.f32_to_bf16_bits(p)
    vs = wl.random_case(8, (1, Hkv, Lk, D), "bf16")
    rng = np.random.default_rng(Lq)
    idx = np.sort(np.stack([rng.choice(Lk, kt, replace=False) for _ in range(H)]), axis=1).astype(np.int32)
    O = torch.full((1, H, Lq, D), 7.0, dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_pv_kmajor(to_device(pt, "bf16", dev)[..., :Lq], to_device(vs, "bf16", dev),
                              torch.from_numpy(idx).to(dev), O, causal=True)
    got = from_device(O)[0]
    V = wl.decode(vs, "bf16").astype(np.float64)[0]
    P = wl.decode(pt, "bf16").astype(np.float64)[0, :, :, :Lq]
    for h in range(H):
        A, Vh = P[h][idx[h]].T, V[h // (H // Hkv)][idx[h]]
        check_product(got[h], A @ Vh, np.abs(A) @ np.abs(Vh), kt, "bf16")


@pytest.mark.parametrize("B,M,K,N,k,wpad", [
    (1, 1, 5, 1, 1, 0),             # 32 x 32 tiles: a single product
    (2, 33, 200, 61, 65, 3),        # partial tiles, one index past a list tile, rows of W unaligned
    (1, 40, 130, 64, 128, 4),       # whole list tiles
    (1, 1025, 96, 1030, 31, 2),     # 64 x 64 tiles: list shorter than a tile, 8-byte rows
    (3, 600, 100, 640, 97, 0),      # ... several units
    (1, 1025, 96, 1029, 31, 3),     # ... 16-byte rows of Y, cut by N
    (2, 17, 20, 50, 16, 2),         # 32 x 32, lists of one tile of 16
    (2, 17, 20, 50, 17, 2),         # ... one index past it
    (64, 32, 40, 130, 33, 0),       # 32 x 32 though 64 x 64 would fill the chip: half empty
    (64, 33, 40, 130, 33, 0),       # ... 64 x 64 one row later
    (64, 33, 40, 130, 15, 1),       # 64 x 64, lists below 16
    (2, 17, 40, 50, 32, 2),         # 32 x 32, lists of one tile of 32
    (128, 100, 40, 20, 17, 0),      # 32 x 32: few columns
])
def test_f32_tiles(B, M, K, N, k, wpad):
    dev = require_gpu()
    xs = wl.random_case(500 + M, (B, M, K), "f32", n_outlier=2)
    ws = wl.random_case(600 + N, (K, N + wpad), "f32", std=0.02)
    rng = np.random.default_rng(M * N)
    idx = np.sort(np.stack([rng.choice(K, k, replace=False) for _ in range(B)]), axis=1).astype(np.int32)
    Y = torch.full((B, M, N + 3), 7.0, dtype=torch.float32, device=dev)
    rmm.rmm_reduced_gemm(to_device(xs, "f32", dev), to_device(ws, "f32", dev)[:, :N], torch.from_numpy(idx).to(dev),
                         Y[:, :, :N])
    got = Y.double().cpu().numpy()
    assert np.all(got[:, :, N:] == 7.0)
    W = ws.astype(np.float64)[:, :N]
    for b in range(B):
        A = xs[b].astype(np.float64)[:, idx[b]]
        check_product(got[b][:, :N], A @ W[idx[b]], np.abs(A) @ np.abs(W[idx[b]]), k, "f32")
