"""fp32 attention with heads of 64 at the sizes where its tiles can go wrong (16 queries a wavefront, 64 queries and 64 keys a
block), and a value that is not finite: only the queries that see it take it."""
import numpy as np
import pytest

import synth
from paper_2504_17449_amd import harness
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_POSTLN, synth.BLOCK_DEC_PRELN])
@pytest.mark.parametrize("lo,hi", [(1, 1), (15, 17), (63, 66), (100, 193)])
def test_fp32_heads_of_64(hmi, block, lo, hi):
    run_case(hmi, small(block, "f32", d_model=128, d_ff=256, n_heads=2, n_tenants=2, hbm_slots=2, n_requests=5, seq_min=lo, seq_max=hi))


@pytest.mark.parametrize("row", [0, 17, 70, 99])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_a_row_that_is_not_finite_stays_unseen_by_earlier_queries(hmi, row, value):
    import torch
    wl = small(synth.BLOCK_DEC_PRELN, "f32", d_model=128, d_ff=256, n_heads=2, n_tenants=1, hbm_slots=1, n_requests=1, seq_min=100,
               seq_max=100)
    ids, lens, x = harness.batch_to_device(wl)
    pool = harness.create_pool(wl)
    try:
        harness.load_tenants(pool, wl)
        y, y_odd = torch.empty_like(x), torch.empty_like(x)
        pool.stack_forward(0, wl.n_layers, x, y, ids, lens)
        x[row, 3] = float(value)
        pool.stack_forward(0, wl.n_layers, x, y_odd, ids, lens)
        torch.cuda.synchronize()
    finally:
        pool.close()
    assert torch.equal(y[:row], y_odd[:row])
    assert not torch.isfinite(y_odd[row:]).all(dim=1).any()


@pytest.mark.parametrize("row", [0, 17, 70, 99])
def test_an_infinite_value_behind_finite_scores(hmi, row):
    """LayerNorm makes a NaN of an infinite input before attention sees it, so here one row's value vector overflows by itself:
    the rows are zero in column 3 after LayerNorm but for one, whose 11 there meets 1e38 in one row of W_v.  W_o does not read
    that column of the context (0 times a number is 0, times an infinity a NaN): earlier queries are as before, later ones are not
    numbers."""
    import torch
    d, n = 128, 100
    wl = small(synth.BLOCK_DEC_PRELN, "f32", d_model=d, d_ff=256, n_heads=2, n_tenants=1, hbm_slots=1, n_requests=1, seq_min=n, seq_max=n)
    ids, lens, x = harness.batch_to_device(wl)
    names = [name for name, _, _ in synth.tensor_specs(wl)]
    w = dict(zip(names, (np.array(t, dtype=np.float32) for t in synth.tenant_tensors(wl, 0, 0))))
    column = 5                                                     # of the second head
    w["wqkv"][:, 3] = 0.0
    w["wqkv"][2 * d + 64 + column, 3] = 1e38
    w["wo"][:, 64 + column] = 0.0
    w["ln1_g"][:], w["ln1_b"][:] = 1.0, 0.0
    x[:, 3] = x[:, torch.arange(d, device=x.device) != 3].mean(dim=1)
    pool = harness.create_pool(wl)
    try:
        pool.load_tenant(0, 0, [w[name] for name in names])
        y, y_odd = torch.empty_like(x), torch.empty_like(x)
        pool.stack_forward(0, 1, x, y, ids, lens)
        x[row] = 0.0
        x[row, 3] = 1.0
        pool.stack_forward(0, 1, x, y_odd, ids, lens)
        torch.cuda.synchronize()
    finally:
        pool.close()
    assert torch.isfinite(y).all()
    assert torch.equal(y[:row], y_odd[:row])
    assert not torch.isfinite(y_odd[row:]).any()
