"""Selection at the edges of its paths (direct ranking of short units, radix
passes that end in a ranked bucket, more ties at the threshold than are
ranked) against the oracle's rule: energy descending, ties to the lower index,
NaN above +inf."""
import numpy as np
import pytest
import torch

import paper_2608_13426_amd as rmm
from tests.gpu_util import gpu, require_gpu

pytestmark = gpu


def _top(e, k):
    v = np.where(np.isnan(e), np.inf, e)
    order = np.lexsort((np.arange(e.size), -v, ~np.isnan(e)))
    return np.sort(order[:k])


def _values(kind, rng, B, K):
    if kind == "ties":                      # a handful of distinct values
        e = rng.integers(0, 3, (B, K)).astype(np.float64)
    elif kind == "zeros":                   # mostly exact zeros, both signs
        e = np.where(rng.random((B, K)) < 0.1, rng.random((B, K)), 0.0) * rng.choice([-0.0, 1.0], (B, K))
    elif kind == "close":                   # equal leading 40 bits, some equal altogether
        e = 1.0 + rng.integers(0, 200, (B, K)) * 2.0 ** -50
    elif kind == "special":
        e = rng.standard_normal((B, K)) ** 2
        e[rng.random((B, K)) < 0.05] = np.inf
        e[rng.random((B, K)) < 0.05] = np.nan
    else:                                   # a bulk within a few percent, 1 % outliers
        e = 1.0 + 0.03 * rng.standard_normal((B, K))
        e[rng.random((B, K)) < 0.01] *= 400.0
    return e


@pytest.mark.parametrize("kind", ["bulk", "ties", "zeros", "close", "special"])
@pytest.mark.parametrize("B,K", [(3, 1), (2, 127), (33, 128), (2, 129), (4, 256), (2, 257), (1, 512), (2, 513),
                                 (1, 2049), (2, 4100), (1, 16385), (1, 33000)])
def test_select_edges(kind, B, K):
    dev = require_gpu()
    rng = np.random.default_rng(K)
    e = _values(kind, rng, B, K)
    for k in sorted({1, (K + 1) // 2, max(1, K - 1), K}):
        idx = torch.full((B * k,), -1, dtype=torch.int32, device=dev)
        rmm.rmm_select(torch.from_numpy(e).to(dev), k, idx)
        got = idx.cpu().numpy().reshape(B, k)
        for b in range(B):
            assert np.array_equal(got[b], _top(e[b], k)), (kind, B, K, k, b)


# one key per thread from 129 to 256 keys; more units than CUs: half as many threads per
# unit up to 512 and from 4097 to 8192 keys, and from 1024 units on up to 1024 keys
@pytest.mark.parametrize("kind", ["bulk", "ties", "zeros", "close", "special"])
@pytest.mark.parametrize("B,K", [(2, 129), (300, 129), (40, 255), (1030, 256), (256, 257), (257, 257),
                                 (300, 512), (256, 4097), (257, 4097), (260, 8192),
                                 (1023, 513), (1024, 513), (1030, 1024)])
def test_select_many_units(kind, B, K):
    dev = require_gpu()
    rng = np.random.default_rng(B + K)
    e = _values(kind, rng, B, K)
    for k in (1, K // 2, K):
        idx = torch.full((B * k,), -1, dtype=torch.int32, device=dev)
        rmm.rmm_select(torch.from_numpy(e).to(dev), k, idx)
        got = idx.cpu().numpy().reshape(B, k)
        for b in range(0, B, max(1, B // 12)):
            assert np.array_equal(got[b], _top(e[b], k)), (kind, B, K, k, b)


# more than 16384 keys: read again, or held in registers (energies, up to 256 units
# of 3e6 keys and more together)
@pytest.mark.parametrize("kind", ["bulk", "ties", "special"])
@pytest.mark.parametrize("B,K", [(1, 32768), (2, 32769), (91, 32768), (92, 32768), (146, 20480), (183, 16400)])
def test_select_wide_units(kind, B, K):
    dev = require_gpu()
    rng = np.random.default_rng(B + K)
    e = _values(kind, rng, B, K)
    for k in (K // 3, K):
        idx = torch.full((B * k,), -1, dtype=torch.int32, device=dev)
        rmm.rmm_select(torch.from_numpy(e).to(dev), k, idx)
        got = idx.cpu().numpy().reshape(B, k)
        for b in range(0, B, max(1, B // 12)):
            assert np.array_equal(got[b], _top(e[b], k)), (kind, B, K, k, b)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,K", [(1, 16385), (3, 32768), (2, 33000)])
def test_select_wide_tokens(dtype, B, K):
    dev = require_gpu()
    g = torch.Generator().manual_seed(K)
    X = torch.randn(B, K + 1, generator=g).to(dtype)
    X[:, ::97] *= 20
    X = X.to(dev)[:, 1:] if dtype == torch.bfloat16 else X.to(dev)[:, :K]     # bf16 off 16-byte boundaries
    e = X.cpu().double().numpy() ** 2
    for k in (1, K // 2):
        idx = torch.full((B * k,), -1, dtype=torch.int32, device=dev)
        rmm.rmm_select_tokens(X, k, idx)
        got = idx.cpu().numpy().reshape(B, k)
        for b in range(B):
            assert np.array_equal(got[b], _top(e[b], k)), (dtype, B, K, k, b)
