"""GELU alone, through the C ABI: a pre-LN decoder with zero attention weights and W1 = 0 gives y = x + W2 GELU(b1) + b2 for every
row x."""
import numpy as np
import pytest
import torch

import synth
from oracle import hmi_oracle as O
from paper_2504_17449_amd import harness
from tests.gemm_rule import kernel
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


# the kernels that have a GELU; the polynomial's error bound holds for -inf as for every x below -4 (the limit is 0), the other
# forms have x Phi(x) = -inf * 0 there
FORMS = [("f32 tiles", "f32", 64, 128, 40, None, False), ("weight stream", "bf16", 256, 256, 3, "stream", False),
         ("tiles, exact form", "bf16", 256, 256, 300, "64x64", False), ("tiles, polynomial", "bf16", 256, 256, 2000, "64x64", True),
         ("persistent tiles", "bf16", 256, 4096, 6500, "persistent", True)]


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("dtype,d,f,rows,want,poly", [c[1:] for c in FORMS], ids=[c[0] for c in FORMS])
def test_one_hidden_value_that_is_not_finite(hmi, dtype, d, f, rows, want, poly, value):
    """One infinity or NaN in the first tenant's b1, W2 = 1: every column of its rows is the sum of GELU(b1); the second tenant's
    three rows know nothing of it."""
    lens = [min(rows, 100)] * (rows // min(rows, 100)) + [3]
    ids = [0] * (len(lens) - 1) + [1]
    assert want is None or kernel(ids, lens, f, d, gelu=True) == want
    b1 = np.zeros((2, f), np.float32)
    b1[0, 5], b1[1, 5] = value, 2.0
    y = activation(dtype, d, f, lens, ids, b1, np.ones((d, f), np.float32))
    with np.errstate(invalid="ignore"):
        gelu = float(O.gelu(np.array([value]))[0])
    if poly and value == -np.inf:
        assert np.abs(y[:-3]).max() <= 2e-4
    else:
        np.testing.assert_array_equal(y[:-3], np.full_like(y[:-3], gelu))
    # 2e-4 of the polynomial, twice half a bf16 unit (the hidden value and the result)
    np.testing.assert_allclose(y[-3:], O.gelu(np.array([2.0]))[0], rtol=2.0 ** -8, atol=2e-4)
