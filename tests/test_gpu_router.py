"""The router at the batch sizes between which its workgroups change (wavefronts, requests per lane, number of workgroups),
with requests on both sides of the length up to which a lane writes their rows by itself."""
import pytest

import synth
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("requests,tenants,seq_max", [
    (1, 1, 9), (64, 7, 9), (65, 65, 20), (256, 3, 8), (257, 100, 40), (512, 300, 70), (513, 40, 12), (1024, 1000, 9), (1025, 5, 30)])
def test_batch_sizes(hmi, requests, tenants, seq_max):
    wl = small(synth.BLOCK_ADAPTER, "bf16", d_model=256, d_ff=64, n_tenants=tenants, hbm_slots=tenants, n_requests=requests,
               seq_min=1, seq_max=seq_max)
    run_case(hmi, wl)
