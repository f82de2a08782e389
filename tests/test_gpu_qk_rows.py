"""The row-streaming reduced QK^T at the edges of its forms (shares of the keys,
rows of S on any element, pieces shifted to lines, gathered dims) against
float64 products: odd lengths, misaligned S, Q and K, Lq != Lk, guards around S."""
import math

import numpy as np
import pytest
import torch

import paper_2608_13426_amd as rmm
import workloads as wl
from tests.gpu_util import check_product, gpu, isclose_inf_pattern, require_gpu, to_device

pytestmark = gpu


def _run(seed, batch, H, Hkv, Lq, Lk, D, k, causal, shift):
    """S written `shift` elements into a guarded buffer, Q and K read `shift` and 2 * `shift`
    elements past a 16-byte boundary; a sample of heads is checked."""
    dev = require_gpu()
    Qs = wl.encode(wl.heavy_tailed_heads((seed, 700), batch * H, Lq, D), "bf16").reshape(batch, H, Lq, D)
    Ks = wl.encode(wl.heavy_tailed_heads((seed, 701), batch * Hkv, Lk, D), "bf16").reshape(batch, Hkv, Lk, D)
    rng = np.random.default_rng(seed)
    idx = np.sort(np.stack([rng.choice(D, k, replace=False) for _ in range(batch * H)]), axis=1).astype(np.int32)
    n = batch * H * Lq * Lk
    qk_in = []
    for i, x in enumerate((Qs, Ks)):                    # off 16-byte boundaries with S
        b = torch.empty(x.size + 8, dtype=torch.bfloat16, device=dev)
        off = (shift * (i + 1)) % 8
        qk_in.append(b[off:off + x.size].view(x.shape))
        qk_in[i].copy_(to_device(x, "bf16", dev))
    buf = torch.full((n + 128,), 7.0, dtype=torch.bfloat16, device=dev)
    S = buf[64 + shift:64 + shift + n].view(batch, H, Lq, Lk)
    rmm.rmm_reduced_qk(*qk_in, torch.from_numpy(idx).to(dev).view(batch, H, k), S, causal=causal)
    assert bool((buf[:64 + shift] == 7.0).all()) and bool((buf[64 + shift + n:] == 7.0).all())
    scale = 1 / math.sqrt(D)
    drop = np.arange(Lk)[None, :] > np.arange(Lq)[:, None] + (Lk - Lq)
    for u in range(0, batch * H, max(1, batch * H // 9)):
        b, h = divmod(u, H)
        A = wl.decode(Qs[b, h], "bf16").astype(np.float64)[:, idx[u]]
        B = wl.decode(Ks[b, h // (H // Hkv)], "bf16").astype(np.float64)[:, idx[u]]
        got = S[b, h].double().cpu().numpy()
        ref = A @ B.T * scale
        mag = np.abs(A) @ np.abs(B).T
        if causal:
            isclose_inf_pattern(got, np.where(drop, -np.inf, ref))
            keep = ~drop
            if not keep.any():
                continue
            got, ref, mag = got[keep], ref[keep], mag[keep]
        check_product(got, ref, mag, k, "bf16", scale)


@pytest.mark.parametrize("batch,H,Hkv,Lq,Lk,D,k,causal,shift", [
    (1, 2, 1, 1, 1, 128, 5, True, 0),           # one score
    (1, 4, 2, 1, 1001, 128, 64, True, 1),       # one query row, key shares, odd rows on odd addresses
    (2, 2, 2, 130, 77, 128, 103, True, 3),      # Lq > Lk: leading rows wholly masked
    (1, 2, 1, 300, 517, 64, 32, False, 0),      # 64 dims, several shares
    (1, 3, 1, 257, 640, 128, 128, True, 0),     # rows on lines, all dims
    (1, 4, 4, 513, 1032, 128, 1, True, 0),      # 16-byte rows, the last share short
    (2, 130, 2, 200, 1411, 128, 90, True, 0),   # long odd rows, below the size at which pieces are shifted
    (1, 512, 4, 7, 1410, 128, 40, False, 5),    # ... even rows on odd addresses, Lk - Lq large
    (1, 300, 2, 129, 1416, 128, 70, True, 0),   # ... 16-byte rows
    (1, 512, 8, 40, 1539, 64, 20, True, 1),     # ... 64 dims
    (1, 1024, 8, 5, 6144, 128, 33, True, 0),    # gathered dims: the longest rows
    (1, 260, 4, 303, 2053, 128, 90, True, 0),   # 320 MB and more: pieces shifted to lines, odd rows
    (1, 256, 4, 322, 2042, 128, 40, False, 5),  # ... every misalignment of even rows
    (1, 250, 2, 316, 2056, 128, 128, True, 0),  # ... 16-byte rows
    (1, 280, 8, 290, 2003, 64, 20, True, 1),    # ... 64 dims
    (1, 256, 4, 304, 2080, 128, 100, True, 0),  # ... every other row at half a line: 256-key tiles
    (1, 256, 4, 304, 2080, 128, 50, False, 0),  # ... gathered
    (1, 48, 2, 1416, 1416, 128, 17, False, 0),  # gathered without the mask
    (2, 60, 4, 1010, 1016, 128, 48, True, 0),   # ... and with it, many blocks
    (1, 48, 8, 1288, 1288, 128, 70, True, 0),   # three shares of the keys, causal
    (1, 23, 23, 300, 900, 64, 64, False, 0),    # one block short of two rounds, 64 dims
])
def test_qk_rows(batch, H, Hkv, Lq, Lk, D, k, causal, shift):
    _run(Lq + Lk, batch, H, Hkv, Lq, Lk, D, k, causal, shift)


@pytest.mark.parametrize("H,Lq,Lk", [(2, 200, 200), (1024, 4, 6144)])
def test_qk_dropped_dims_have_no_effect(H, Lq, Lk):
    """Infinite and NaN values in dims outside the set leave S unchanged."""
    dev = require_gpu()
    g = torch.Generator(device=dev).manual_seed(1)
    Q = torch.randn(1, H, Lq, 128, device=dev, generator=g).bfloat16()
    K = torch.randn(1, 2, Lk, 128, device=dev, generator=g).bfloat16()
    idx = torch.arange(0, 128, 2, dtype=torch.int32, device=dev).repeat(H).view(1, H, 64)
    S, T = torch.empty(2, 1, H, Lq, Lk, dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_qk(Q, K, idx, S)
    Q[..., 1], Q[..., 3], K[..., 1], K[..., 5] = math.inf, math.nan, math.nan, -math.inf
    rmm.rmm_reduced_qk(Q, K, idx, T)
    assert torch.equal(S.view(torch.int16), T.view(torch.int16))
