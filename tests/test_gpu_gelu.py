"""GELU alone, through the C ABI: a pre-LN decoder with zero attention weights and W1 = 0 gives y = x + W2 GELU(b1) + b2 for every
row x."""
import numpy as np
import pytest
import torch

import synth
from oracle import hmi_oracle as O
from paper_2504_17449_amd import harness
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu


def activation(dtype, d, f, lens, ids, b1, w2):
    """y [rows, d] for x = 0, one layer, the tenants' b1 [tenant][f] and one W2 [d, f]."""
    wl = small(synth.BLOCK_DEC_PRELN, dtype, d_model=d, d_ff=f, n_heads=d // 64, n_tenants=len(b1), hbm_slots=len(b1))
    zeros = lambda *shape: np.zeros(shape, np.float32)
    pool = harness.create_pool(wl, max_requests=len(lens), max_tokens=sum(lens))
    try:
        for t in range(len(b1)):
            w = {"wqkv": zeros(3 * d, d), "bqkv": zeros(3 * d), "wo": zeros(d, d), "bo": zeros(d), "ln1_g": zeros(d) + 1,
                 "ln1_b": zeros(d), "w1": zeros(f, d), "b1": b1[t], "w2": w2, "b2": zeros(d), "ln2_g": zeros(d) + 1, "ln2_b": zeros(d)}
            pool.load_tenant(t, 0, [synth.to_storage_bytes(w[n], dtype) for n, _, _ in synth.tensor_specs(wl)])
        x = torch.zeros(sum(lens), d, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        y = torch.empty_like(x)
        pool.forward(0, x, y, ids, lens)
        torch.cuda.synchronize()
    finally:
        pool.close()
    return y.double().cpu().numpy()


@pytest.mark.parametrize("spread", [0.16, 0.3, 0.55, 1.0])
def test_fp32_hidden_values_of_the_usual_size(hmi, spread):
    """1 024 hidden values N(0, spread) of an fp32 pool.  x Phi(x) by erf has four roundings (x / sqrt 2, erf, 1 + erf, the
    product), each with the error of rounding the result once or less: together twice that, and a tenth for erf's own."""
    d = 256
    b1 = (np.random.default_rng(3).standard_normal((4, d)) * spread).astype(np.float32)
    y = activation("f32", d, d, [1] * 4, list(range(4)), b1, np.eye(d, dtype=np.float32))
    want = O.gelu(b1.astype(np.float64))
    once = np.linalg.norm(want.astype(np.float32) - want)
    print(f"  spread {spread}: error {np.linalg.norm(y - want) / np.linalg.norm(want):.2e}, rounded once {once / np.linalg.norm(want):.2e}", flush=True)
    assert np.linalg.norm(y - want) <= 2.2 * once
