"""The attention block for a few query rows (a decode step) against the oracle:
edges of its key tiles, head groups and key splits, and both output forms."""
import math

import numpy as np
import pytest
import torch

import paper_2608_13426_amd as rmm
import workloads as wl
from oracle import rmm_oracle as ro
from tests.gpu_util import attention_bound, check_energies, from_device, gpu, require_gpu, to_device

pytestmark = gpu

D = 128


def _inputs(seed, b, H, Hkv, Lq, Lk, r):
    Qs = wl.encode(wl.heavy_tailed_heads((seed, 500), b * H, Lq, D), "bf16").reshape(b, H, Lq, D)
    Ks = wl.encode(wl.heavy_tailed_heads((seed, 501), b * Hkv, Lk, D), "bf16").reshape(b, Hkv, Lk, D)
    Vs = wl.random_case(seed + 502, (b, Hkv, Lk, D), "bf16")
    Q = wl.decode(Qs, "bf16").astype(np.float64)
    k = ro.retained_count(r, D)
    idx = np.stack([np.stack([ro.topk_indices(ro.column_energies(Q[i, h]), k) for h in range(H)])
                    for i in range(b)]).astype(np.int32)
    return Qs, Ks, Vs, idx


def _check(O, Qs, Ks, Vs, idx, causal, scale=None):
    Q, K, V = (wl.decode(x, "bf16").astype(np.float64) for x in (Qs, Ks, Vs))
    s = D ** -0.5 if scale is None else float(np.float32(scale))
    for i in range(Q.shape[0]):
        ref = ro.reduced_attention(Q[i] * (s * math.sqrt(D)), K[i], V[i], idx[i], causal)
        bound = attention_bound(Q[i], K[i], V[i], idx[i], causal, s)
        assert np.all(np.abs(O[i] - ref) <= bound[:, :, None] + 2.0 ** -8 * np.abs(ref))


@pytest.mark.parametrize("b,H,Hkv,Lq,Lk,r,causal,scale", [
    (1, 1, 1, 1, 9, 0.25, True, None),        # one head, one short tile
    (2, 4, 4, 1, 129, 0.5, True, None),       # one head per kv head: 128-key stages, tail of one key
    (1, 4, 2, 3, 700, 0.5, True, -0.05),      # pairs; negative scale; several splits
    (1, 6, 2, 2, 333, 0.8, True, None),       # three heads per kv head (one wave idle)
    (1, 8, 1, 16, 1500, 1.0, True, None),     # eight heads, all 16 rows
    (1, 20, 2, 5, 260, 0.001, False, 0.0),    # ten heads per kv head: two chunks; k = 1; zero scale
    (2, 4, 1, 13, 300, 0.5, False, 3.0),      # large scores: the maximum rises several times
    (1, 4, 2, 15, 9, 0.25, True, None),       # more queries than keys (the prefill kernel): leading rows are zero
    (1, 2, 1, 17, 200, 0.5, True, None),      # two blocks of query rows, the second of one
    (1, 4, 1, 70, 900, 0.8, True, None),      # five, several splits
    (1, 4, 1, 256, 600, 1.0, True, None),     # causal: the last split is wholly masked for the early rows
    (1, 4, 2, 224, 530, 1.0, True, None),     # ... pairs: and for some key tiles of a stage
    (1, 2, 2, 200, 470, 1.0, True, None),     # ... one head per kv head
])
def test_few_rows(b, H, Hkv, Lq, Lk, r, causal, scale):
    dev = require_gpu()
    Qs, Ks, Vs, idx = _inputs(Lk, b, H, Hkv, Lq, Lk, r)
    O = torch.full((b, H, Lq, D), 3.0, dtype=torch.bfloat16, device=dev)
    args = [to_device(x, "bf16", dev) for x in (Qs, Ks, Vs)] + [torch.from_numpy(idx).to(dev)]
    rmm.rmm_reduced_attention(*args, O, causal=causal, scale=scale)
    _check(from_device(O), Qs, Ks, Vs, idx, causal, scale)
    O2 = torch.empty_like(O)
    rmm.rmm_reduced_attention(*args, O2, causal=causal, scale=scale)
    assert torch.equal(O.view(torch.int16), O2.view(torch.int16))


@pytest.mark.parametrize("b,H,Hkv,Lq,Lk", [(2, 8, 2, 8, 600), (1, 4, 4, 16, 150), (1, 2, 1, 8, 40),
                                           (1, 4, 1, 256, 1300), (1, 4, 2, 248, 1100), (1, 2, 2, 200, 900),
                                           # many heads: the merge's other forms
                                           (64, 8, 2, 8, 120), (64, 8, 4, 32, 300), (96, 16, 4, 24, 250),
                                           (192, 8, 2, 8, 70), (96, 16, 4, 16, 200)])
def test_few_rows_kmajor_same_bits(b, H, Hkv, Lq, Lk):
    """The K-major form holds the plain block's values bit for bit, with their energies."""
    dev = require_gpu()
    Qs, Ks, Vs, idx = _inputs(Lk, b, H, Hkv, Lq, Lk, 0.5)
    args = [to_device(x, "bf16", dev) for x in (Qs, Ks, Vs)] + [torch.from_numpy(idx).to(dev)]
    O = torch.empty((b, H, Lq, D), dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_attention(*args, O)
    Ot = torch.full((b, H * D, Lq + 8), 7.0, dtype=torch.bfloat16, device=dev)
    e = torch.empty((b, H * D), dtype=torch.float64, device=dev)
    rmm.rmm_reduced_attention_kmajor(*args, Ot, e)
    want = O.permute(0, 1, 3, 2).reshape(b, H * D, Lq)
    assert torch.equal(Ot[:, :, :Lq].contiguous().view(torch.int16), want.contiguous().view(torch.int16))
    assert bool((Ot[:, :, Lq:] == 7.0).all())
    x = from_device(want)
    for i in range(b):
        check_energies(e[i].cpu().numpy(), (x[i] ** 2).sum(1), Lq)


def test_few_rows_ignore_nonfinite_dropped_dims():
    """Infinite and NaN key or query values in dims outside a head's set have no effect."""
    dev = require_gpu()
    Qs, Ks, Vs, idx = _inputs(3, 1, 4, 2, 2, 300, 0.5)
    shared = [sorted(set(range(D)) - set(idx[0, 2 * g].tolist()) - set(idx[0, 2 * g + 1].tolist())) for g in range(2)]
    args = [to_device(x, "bf16", dev) for x in (Qs, Ks, Vs)] + [torch.from_numpy(idx).to(dev)]
    O = torch.empty((1, 4, 2, D), dtype=torch.bfloat16, device=dev)
    rmm.rmm_reduced_attention(*args, O)
    assert all(shared)
    for g in range(2):
        args[1][0, g, ::3, shared[g][0]] = math.inf
        args[1][0, g, 1::3, shared[g][-1]] = math.nan
        args[0][0, 2 * g, :, shared[g][0]] = math.nan
    O2 = torch.empty_like(O)
    rmm.rmm_reduced_attention(*args, O2)
    assert torch.equal(O.view(torch.int16), O2.view(torch.int16))


@pytest.mark.parametrize("H,Hkv,Lq,Lk", [(4, 1, 64, 400), (4, 2, 128, 700), (2, 2, 48, 300), (8, 1, 17, 200)])
def test_few_rows_causal_future_values(H, Hkv, Lq, Lk):
    """Non-finite value and key rows after a 16-row block's last visible key have no effect on the block."""
    dev = require_gpu()
    Qs, Ks, Vs, idx = _inputs(7, 1, H, Hkv, Lq, Lk, 0.5)
    args = [to_device(x, "bf16", dev) for x in (Qs, Ks, Vs)] + [torch.from_numpy(idx).to(dev)]
    O, O2 = (torch.empty((1, H, Lq, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
    rmm.rmm_reduced_attention(*args, O)
    for q0 in range(0, Lq - 16, 16):
        first = q0 + 16 + Lk - Lq
        args[1][:, :, first:], args[2][:, :, first::2], args[2][:, :, first + 1::2] = math.nan, math.inf, math.nan
        rmm.rmm_reduced_attention(*args, O2)
        rows = slice(q0, q0 + 16)
        assert torch.equal(O[:, :, rows].contiguous().view(torch.int16), O2[:, :, rows].contiguous().view(torch.int16))
        for x, y in zip((1, 2), (Ks, Vs)):
            args[x] = to_device(y, "bf16", dev)
