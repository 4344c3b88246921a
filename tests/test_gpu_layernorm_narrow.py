"""LayerNorm of rows that are no multiple of 256 wide: as many columns a lane as there are where the width is a multiple of 64, the
general form for the others (fp32), over rows that leave wavefronts of the last workgroup without one, with the tenants' own and with
shared parameters."""
import pytest

import synth
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128, 192, 320, 384])
@pytest.mark.parametrize("block,dtype", [(synth.BLOCK_ENC_POSTLN, "f32"), (synth.BLOCK_ENC_POSTLN, "bf16"),
                                         (synth.BLOCK_DEC_PRELN, "bf16"), (synth.BLOCK_DEC_ADAPTER, "bf16")])
@pytest.mark.parametrize("tenants,requests,lo,hi", [(1, 1, 1, 1), (3, 3, 1, 3), (40, 60, 2, 5)])
def test_narrow_rows(hmi, d, block, dtype, tenants, requests, lo, hi):
    wl = small(block, dtype, d_model=d, d_ff=4 * d, n_heads=d // 64, n_layers=1, n_tenants=tenants, hbm_slots=tenants,
               n_requests=requests, seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))


@pytest.mark.parametrize("dtype,d", [(dtype, d) for d in (448, 576, 640, 704, 832, 896, 960, 1088, 1280, 1984) for dtype in ("f32", "bf16")]
                         + [("f32", d) for d in (16, 80, 336, 1040, 2032)])
def test_odd_widths(hmi, dtype, d):
    """Every other width a lane, and fp32 widths that are no multiple of 64: 1, 2 and 3 rows of the last workgroup."""
    for requests in (1, 6, 11):
        wl = small(synth.BLOCK_FFN, dtype, d_model=d, d_ff=64, n_layers=1, n_tenants=5, hbm_slots=5, n_requests=requests, seq_min=1, seq_max=1)
        run_case(hmi, wl)
