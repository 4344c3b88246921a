"""The GEMM of a few rows through shared weights: units of k that fill the wavefronts once, partly, twice and three times, halves of a
column block where k is short, one row to one past a block of 4, 8 and 16, several row blocks, and columns that leave XCDs without any."""
import ctypes as C

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import run_case, small

BLOCKS = [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER]
CASES = [      # d, f, requests, lengths
    (128, 128, 1, 1, 1), (128, 1664, 1, 4, 4), (256, 512, 1, 5, 5), (256, 3200, 2, 4, 4), (384, 896, 2, 2, 3),
    (768, 3072, 3, 3, 3), (768, 3072, 1, 16, 16), (768, 3072, 1, 17, 17), (768, 3072, 2, 33, 40),
    (1024, 4096, 1, 6, 6), (1024, 4608, 2, 1, 3), (512, 2048, 1, 1, 1),
]


def thin(rows, n_out, k, gelu=False, n_cu=256):
    import paper_2504_17449_amd as hmi
    fn = hmi.lib.hmi_internal_gemm_thin
    fn.restype, fn.argtypes = C.c_int32, [C.c_int32] * 5
    return bool(fn(rows, n_out, k, gelu, n_cu))


def launches(d, f):
    return (3 * d, d, False), (d, d, False), (f, d, True), (d, f, False)


def test_rule():
    rng = np.random.default_rng(0)
    for _ in range(4000):
        rows, n_out, k, n_cu = int(rng.integers(1, 400)), 16 * int(rng.integers(1, 300)), 64 * int(rng.integers(1, 90)), int(rng.choice([256, 64]))
        gelu = bool(rng.integers(0, 2))
        if thin(rows, n_out, k, gelu, n_cu):     # whole units of k, at most three a wavefront; a round of workgroups, or two
            assert k % 128 == 0 and k <= 36 * 128
            assert -(-rows // 16) * (n_out // 16) <= n_cu * (2 if gelu and k <= 768 else 1)
    units = set()
    for d, f, requests, lo, hi in CASES:
        assert any(thin(requests * lo, *size) for size in launches(d, f))
        units |= {size[1] // 128 for size in launches(d, f) if thin(requests * hi, *size)}
    assert {1, 2, 4, 6, 8, 13, 24, 25, 36} <= units
    # sizes that other tests mean for the forms behind this rule
    assert not thin(33, 2304, 768) and not thin(33, 3072, 768, True) and not thin(256, 768, 3072) and not thin(141, 768, 768)


@pytest.mark.gpu
@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("d,f,requests,lo,hi", CASES)
def test_a_few_rows_of_shared_weights(hmi, block, d, f, requests, lo, hi):
    wl = small(block, "bf16", d_model=d, d_ff=f, n_heads=d // 64, n_layers=1, n_tenants=2, hbm_slots=2, n_requests=requests, seq_min=lo,
               seq_max=hi)
    run_case(hmi, wl)
