"""The adapter kernel that also normalises its rows (shared layers, rank 64), at every width it takes: a few rows of each
tenant (units of 32 rows that are nearly empty), and enough rows that a workgroup walks several units and tenants."""
import pytest

import synth
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
@pytest.mark.parametrize("d", [256, 512, 768])
@pytest.mark.parametrize("layers,tenants,requests,lo,hi", [(1, 9, 9, 1, 3), (2, 5, 12, 31, 97), (1, 7, 90, 150, 333)])
def test_adapted_rows_normalised(hmi, block, d, layers, tenants, requests, lo, hi):
    wl = small(block, "bf16", d_model=d, d_ff=512, n_heads=d // 64, n_layers=layers, n_tenants=tenants, hbm_slots=tenants,
               n_requests=requests, seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))
