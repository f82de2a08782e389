"""Row statistics of the attention weights at the edges of a row group's batches
(16 or 64 lanes of eight 16-byte loads: 1024 or 4096 keys), with fully masked and
all -inf rows, against float64 softmax."""
import numpy as np
import pytest
import torch

import paper_2608_13426_amd as rmm
from tests.gpu_util import U16, gpu, require_gpu

pytestmark = gpu


@pytest.mark.parametrize("U,Lq,Lk,causal", [
    (1, 1, 1, True), (3, 5, 7, False), (2, 17, 8, True), (1, 40, 129, True), (1, 3, 1024, False),
    (2, 9, 1025, False), (1, 20, 1040, True), (1, 2100, 2050, True),
    (3, 701, 1025, True), (5, 420, 1031, False),     # 16 lanes per row, second batch of a few keys
    (2, 3, 4097, False), (1, 33, 4101, True), (7, 1, 513, True),    # a wave per row, one batch and two
])
def test_weights_row_statistics(U, Lq, Lk, causal):
    dev = require_gpu()
    rng = np.random.default_rng(Lk)
    ld = (Lk + 7) // 8 * 8
    s = 4.0 * rng.standard_normal((U, Lq, Lk)) + 30.0 * rng.standard_normal((U, Lq, 1))
    s[:, Lq // 2, :] = -np.inf
    S = torch.full((1, U, Lq, ld), float("nan"), dtype=torch.bfloat16, device=dev)    # NaN past Lk
    S[0, :, :, :Lk] = torch.from_numpy(s).to(dev).bfloat16()
    ldt = (Lq + 7) // 8 * 8
    Pt = torch.zeros(1, U, Lk, ldt, dtype=torch.bfloat16, device=dev)
    e = torch.empty(U * Lk, dtype=torch.float64, device=dev)
    rmm.rmm_attention_weights_kmajor(S[..., :Lk], Pt[..., :Lq], e, causal=causal)
    x = S[0, :, :, :Lk].double().cpu().numpy()
    if causal:
        x = np.where(np.arange(Lk)[None, :] > np.arange(Lq)[:, None] + (Lk - Lq), -np.inf, x)
    m = x.max(axis=-1, keepdims=True)
    p = np.exp(x - np.where(np.isfinite(m), m, 0.0))
    tot = p.sum(axis=-1, keepdims=True)
    p = np.where(tot > 0, p / np.where(tot > 0, tot, 1.0), 0.0)
    got = Pt[0, :, :, :Lq].double().cpu().numpy().transpose(0, 2, 1)
    # one rounding to bf16 (8 significand bits: at most 2^-8 = U16 relative), and
    # fp32 errors of the exponential (a few units of the score difference) and of
    # the row's sum
    far = np.where(np.isfinite(x), np.abs(x - np.where(np.isfinite(m), m, 0.0)), 0.0)
    assert np.all(np.abs(got - p) <= p * (U16 + 2.0 ** -20 * (1 + far)) + 2.0 ** -130)
