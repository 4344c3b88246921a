"""Sums of fp32 products: no further from 64 bits than one chain of fused multiply-adds in fp32 is."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_17449_amd import harness
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [64, 80, 256, 768])
def test_products_of_an_fp32_pool(hmi, k):
    """An adapter whose up-projection is the identity: y = x + ReLU(W x), W some thousand times x, so that y's error is that of
    the sum over k.  The chain has k roundings of partial sums that grow; two chains of half as many terms have 0.7 of its error
    (0.8 at k = 64 with the roundings at the end); one chain of matrix products has 1.00 to 1.01."""
    rows, r = 1024, 64
    rng = np.random.default_rng(k)
    x = rng.standard_normal((rows, k)).astype(np.float32)
    w = (rng.standard_normal((r, k)) * 3000).astype(np.float32)
    wl = small(synth.BLOCK_ADAPTER, "f32", d_model=k, d_ff=r, n_tenants=1, hbm_slots=1)
    up = np.zeros((k, r), np.float32)
    up[:r] = np.eye(r)
    pool = harness.create_pool(wl, max_requests=8, max_tokens=rows)
    try:
        t = {"w_down": w, "b_down": np.zeros(r, np.float32), "w_up": up, "b_up": np.zeros(k, np.float32)}
        names = [n for n, _, _ in synth.tensor_specs(wl)]
        pool.load_tenant(0, 0, [t[n] for n in names])
        xd = torch.from_numpy(x).cuda()
        y = torch.empty_like(xd)
        pool.forward(0, xd, y, [0] * 8, [rows // 8] * 8)
        torch.cuda.synchronize()
    finally:
        pool.close()
    chain = np.zeros((rows, r), np.float32)
    for i in range(k):       # one rounding a step: the product of two floats is exact in 64 bits (and its sum with a third nearly so)
        chain = (chain + x[:, i:i + 1].astype(np.float64) * w[:, i].astype(np.float64)).astype(np.float32)
    chain = np.maximum(chain, 0) + x[:, :r]
    want = np.maximum(x.astype(np.float64) @ w.astype(np.float64).T, 0) + x[:, :r]
    got = np.linalg.norm(y.cpu().numpy()[:, :r] - want) / np.linalg.norm(want)
    bar = np.linalg.norm(chain - want) / np.linalg.norm(want)
    print(f"  k = {k}: {got:.3e}, one chain {bar:.3e}, ratio {got / bar:.3f}", flush=True)
    assert got <= 0.9 * bar
