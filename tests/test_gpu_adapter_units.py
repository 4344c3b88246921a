"""The adapter kernel where the size of its units changes: units of 8, 16 and 32 rows (the smallest of which there is one for
each compute unit at most), one more than that, and more tenants than are counted exactly."""
import numpy as np
import pytest
import torch

import synth
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu

RANK = 64


def _adapter(hmi, d, rows):
    """rows[t]: rows of tenant t, one request each; every row against float64, adapters that make up most of the result."""
    rng = np.random.default_rng(d + sum(rows))
    tenants, n = len(rows), sum(rows)

    def bf16(*shape, scale):
        return torch.from_numpy(rng.standard_normal(shape) * scale).to(torch.bfloat16)

    weights = [(bf16(RANK, d, scale=0.1), bf16(RANK, scale=0.5), bf16(d, RANK, scale=0.2), bf16(d, scale=0.5)) for _ in range(min(tenants, 9))]
    order = rng.permutation(tenants).astype(np.int32)
    lens = np.array([rows[t] for t in order], dtype=np.int32)
    x = bf16(n, d, scale=1.0)
    pool = hmi.Pool(block=hmi.HMI_BLOCK_ADAPTER, dtype=hmi.HMI_BF16, d_model=d, d_ff=RANK, n_heads=0, n_layers=1, max_tenants=tenants,
                    hbm_slots=tenants, host_tier=False, max_requests=tenants, max_tokens=n, ln_eps=1e-12,
                    compute_stream=torch.cuda.current_stream().cuda_stream, adapter_rank=RANK, max_classes=0)
    try:
        for t in range(tenants):
            pool.load_tenant(t, 0, [w.view(torch.int16).numpy().view(np.uint16) for w in weights[t % len(weights)]])
        y = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        pool.stack_forward(0, 1, x.cuda(), y, order, lens)
        torch.cuda.synchronize()
    finally:
        pool.close()
    got, at = y.double().cpu(), 0
    for t, length in zip(order, lens):
        wd, bd, wu, bu = (w.double() for w in weights[t % len(weights)])
        xs = x[at:at + length].double()
        a = torch.relu(xs @ wd.T + bd) @ wu.T + bu
        # one rounding of the bottleneck (2^-9 of each of its 64 values, random signs) and one of the result
        bound = 2.0 ** -8 * (a.abs() + xs.abs()) + 6 * 2.0 ** -9 * (torch.relu(xs @ wd.T + bd) ** 2 @ wu.T ** 2).sqrt() + 1e-3
        off = (got[at:at + length] - xs - a).abs()
        assert bool((off <= bound).all()), (int(t), int(length), float((off / bound).max()))
        at += length


@pytest.mark.parametrize("d", [256, 768])
@pytest.mark.parametrize("rows", [
    [1], [8], [9], [33, 1, 16, 17, 7],
    [2048], [2041, 1],                 # 256 + 1 units of eight: 16 rows a unit
    [2049], [4096],                    # 257 of eight; 256 of sixteen
    [4097], [8192], [8193],            # 32 rows; 256 units; one more than there are compute units
    [1] * 255 + [9],                   # 256 tenants, 257 units of eight
    [1] * 256, [1] * 257, [3] * 300,   # as many tenants as are counted exactly, and more
])
def test_units_of_the_adapter(hmi, d, rows):
    _adapter(hmi, d, rows)


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
@pytest.mark.parametrize("tenants,requests,lo,hi", [(4, 4, 7, 17), (2, 9, 300, 340), (3, 30, 190, 200), (260, 300, 1, 2)])
def test_units_of_the_adapter_with_its_norm(hmi, block, tenants, requests, lo, hi):
    """Units of 8, 16, 32 rows and the general form, in front of the layer's LayerNorm (two layers: its other input is fp32 in the second)."""
    wl = small(block, "bf16", d_model=768, d_ff=512, n_heads=12, n_layers=2, n_tenants=tenants, hbm_slots=tenants,
               n_requests=requests, seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))
