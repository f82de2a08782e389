"""Shared decode products where a product workgroup takes a run of several
ranges (the last run short, empty ranges inside), against float64 products."""
import pytest
import torch

import paper_2608_13426_amd as rmm
from tests.gpu_util import U16, U32, gpu, require_gpu

pytestmark = gpu


@pytest.mark.parametrize("B,K,N,k", [
    (16, 2600, 17200, 1300),     # 408 workgroups at one range each: runs of two
    (8, 2600, 35000, 700),       # 822: runs of four, the last of two ranges
    (32, 512, 205000, 300),      # one range only: Y written directly
    (9, 2600, 22000, 1300),      # 516: runs of four
    (3, 2600, 17200, 2600),      # narrow tiles: 810, runs of two, all rows kept
    (5, 2600, 22000, 1000),      # ... 1032: one range each
    (7, 2600, 44000, 500),       # ... 2064: runs of two
    (2, 2600, 128008, 200),      # ... 6006, runs of four
])
def test_runs(B, K, N, k):
    dev = require_gpu()
    g = torch.Generator(device=dev).manual_seed(K + B)
    X = torch.randn(B, K, device=dev, generator=g).bfloat16()
    W = (0.02 * torch.randn(K, N, device=dev, generator=g)).bfloat16()
    lo = 600 if k < 1000 else 0                      # a whole range without kept rows
    idx = torch.stack([torch.sort(lo + torch.randperm(K - lo, device=dev, generator=g)[:k]).values
                       if K > 600 else torch.sort(torch.randperm(K, device=dev, generator=g)[:k]).values
                       for _ in range(B)]).int().contiguous()
    Y = torch.full((B, N), 7.0, dtype=torch.bfloat16, device=dev)
    rmm.rmm_decode_products_shared([(X, W, k, idx.view(-1), Y)])
    for b in range(B):
        x, w = X[b][idx[b].long()].double(), W[idx[b].long()].double()
        ref, mag = x @ w, x.abs() @ w.abs()
        # fp32 sums of k exact products in any order, one rounding to bf16
        tol = U16 * ref.abs() + (k + 2) * U32 * mag * (1 + U16)
        assert bool(((Y[b].double() - ref).abs() <= tol).all()), b
