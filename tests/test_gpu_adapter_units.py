"""The adapter kernel where the size of its units changes: the smallest units of 8, 16 (in front of a LayerNorm only) and 32 rows of
which there is one for each compute unit at most, the general form for one more than that and for more tenants than are counted
exactly.  Every case asserts which units the launcher's rule gives it."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_17449_amd import harness
from tests.gemm_rule import adapter_unit
from tests.oracle_side import compare, oracle_forward, rows_of
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
@pytest.mark.parametrize("rows,unit", [
    ([1], 8), ([8], 8), ([9], 8), ([33, 1, 16, 17, 7], 8),
    ([2048], 8), ([2041, 1], 32),               # 256 units of eight, and 257: without a LayerNorm the next larger ones have 32 rows
    ([2049], 32), ([4096], 32), ([4097], 32),
    ([8192], 32), ([8193], 0),                  # 256 units of 32; one more than there are compute units
    ([1] * 255 + [9], 32),                      # 256 tenants, 257 units of eight
    ([1] * 256, 8), ([1] * 257, 0), ([3] * 300, 0),   # as many tenants as are counted exactly, and more
])
def test_units_of_the_adapter(hmi, d, rows, unit):
    assert adapter_unit(rows, False) == unit
    _adapter(hmi, d, rows)


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
@pytest.mark.parametrize("tenants,requests,lo,hi,unit", [(4, 4, 7, 17, 8), (2, 9, 300, 340, 16), (3, 30, 190, 200, 32), (260, 300, 1, 2, 8)])
def test_units_of_the_adapter_with_its_norm(hmi, block, tenants, requests, lo, hi, unit):
    """In front of the layer's LayerNorm, long requests too (two layers: the LayerNorm's other input is fp32 in the second)."""
    wl = small(block, "bf16", d_model=768, d_ff=512, n_heads=12, n_layers=2, n_tenants=tenants, hbm_slots=tenants,
               n_requests=requests, seq_min=lo, seq_max=hi)
    ids, lens = synth.batch_ids_lens(wl)
    assert adapter_unit([int(lens[ids == t].sum()) for t in np.unique(ids)], True) == unit
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))


LONGEST = 61          # rows of a request below, at most


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
@pytest.mark.parametrize("d", [256, 768])
@pytest.mark.parametrize("rows,unit", [
    ([2048], 8), ([2041, 1], 16), ([2049], 16),     # 256 units of eight; 257: units of 16, the last of one row
    ([4096], 16), ([4081, 1], 32), ([4097], 32),    # 256 units of 16; 257
    ([8192], 32), ([8193], 0),                      # 256 units of 32; 257: workgroups with several
    ([1] * 256, 8), ([1] * 255 + [9], 16),          # 256 tenants
    ([1] * 257, 0), ([1, 2, 3] * 100, 0),           # more: the general form, whose workgroups change tenants from unit to unit
])
def test_limits_of_the_units_with_their_norm(hmi, block, d, rows, unit):
    """rows[t]: rows of tenant t, in requests of up to LONGEST, in random order; the requests at both ends of the sorted batch, of the
    largest tenant and of some others against float64."""
    assert adapter_unit(rows, True) == unit
    rng = np.random.default_rng(len(rows) + sum(rows))
    pieces = [(t, min(LONGEST, n - at)) for t, n in enumerate(rows) for at in range(0, n, LONGEST)]
    ids, lens = np.array([pieces[i] for i in rng.permutation(len(pieces))], dtype=np.int32).T.copy()
    tenants, n = len(rows), int(lens.sum())
    wl = small(block, "bf16", d_model=d, d_ff=256, n_heads=d // 64, n_layers=2, n_tenants=tenants, hbm_slots=tenants,
               n_requests=len(ids), seq_min=1, seq_max=LONGEST)
    order = np.argsort(ids, kind="stable")
    biggest = order[ids[order] == int(np.argmax(rows))]
    sample = sorted({int(r) for r in (*order[:2], *order[-2:], biggest[0], biggest[-1], *rng.integers(0, len(ids), 6))})
    x = harness.host_to_device(np.concatenate([synth.hidden_states(wl, r, int(lens[r]), 0) for r in range(len(ids))]), "bf16")
    pool = harness.create_pool(wl, max_requests=len(ids), max_tokens=n)
    try:
        harness.load_tenants(pool, wl)
        y = torch.empty_like(x)
        pool.stack_forward(0, 2, x, y, ids, lens)
        torch.cuda.synchronize()
        got = harness.device_to_f64(y)
    finally:
        pool.close()
    assert np.isfinite(got).all()
    max_abs, rel, ok = compare(got, oracle_forward(wl, ids, lens, sample), rows_of(lens, sample), "bf16")
    assert ok, (max_abs, rel)
