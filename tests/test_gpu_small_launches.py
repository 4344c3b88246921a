"""GEMM launches of a round of workgroups or less: tiles of 32 x 32 to 128 x 64 with one and two lines of k a stage, the split of
shared weights' tiles among the XCDs, and k shared by four wavefronts, at single rows, one row past a block of 8 or a tile, and widths
that leave XCDs without tiles."""
import pytest

import synth
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
@pytest.mark.parametrize("d,f,requests,lo,hi", [
    (768, 3072, 1, 1, 1), (768, 3072, 1, 8, 8), (768, 3072, 3, 3, 3), (768, 3072, 2, 16, 17),     # 1, 8, 9, 33 rows
    (768, 3072, 2, 40, 101), (768, 3072, 2, 128, 128), (768, 3072, 5, 61, 61),                    # 141, 256, 305 rows
    (768, 3072, 7, 16, 200), (768, 3072, 19, 70, 70),                                             # 756, 1 330 rows
    (512, 2048, 3, 20, 31), (256, 1024, 4, 33, 33),
    (320, 1280, 2, 30, 41), (64, 256, 1, 17, 17), (192, 768, 3, 60, 70),                          # k an odd number of lines
])
def test_shared_weights(hmi, block, d, f, requests, lo, hi):
    wl = small(block, "bf16", d_model=d, d_ff=f, n_heads=d // 64, n_layers=1, n_tenants=3, hbm_slots=3, n_requests=requests,
               seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))


@pytest.mark.parametrize("block,heads", [(synth.BLOCK_FFN, 0), (synth.BLOCK_ENC_POSTLN, 1), (synth.BLOCK_DEC_PRELN, 1)])
@pytest.mark.parametrize("d,f,tenants,requests,lo,hi", [
    (768, 3072, 1, 1, 33, 33), (768, 3072, 1, 1, 40, 40), (768, 1024, 2, 4, 64, 65), (512, 2048, 1, 5, 100, 110),
    (320, 1280, 2, 3, 50, 90), (128, 512, 3, 9, 60, 60), (1024, 4096, 1, 2, 90, 100),
])
def test_a_tenants_own_weights(hmi, block, heads, d, f, tenants, requests, lo, hi):
    wl = small(block, "bf16", d_model=d, d_ff=f, n_heads=heads * d // 64, n_layers=1, n_tenants=tenants, hbm_slots=tenants,
               n_requests=requests, seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))


@pytest.mark.parametrize("d,f,tenants,requests,lo,hi", [
    (64, 128, 1, 1, 1, 1), (64, 192, 3, 3, 31, 33), (128, 512, 2, 4, 64, 65), (192, 768, 2, 3, 40, 70),     # k = 64, 128, 192
    (320, 1280, 1, 2, 33, 33), (512, 2048, 3, 5, 20, 90), (768, 3072, 1, 1, 1, 1), (768, 3072, 2, 3, 60, 130),
    (512, 2048, 4, 40, 100, 128), (768, 3072, 5, 30, 64, 64), (768, 3072, 2, 90, 65, 65),                   # several rounds
])
def test_fp32_tiles(hmi, d, f, tenants, requests, lo, hi):
    """32 x 32 with k in four parts, 64 x 32 with k in two, 64 x 64: single rows, one row past a tile, one and several rounds."""
    wl = small(synth.BLOCK_FFN, "f32", d_model=d, d_ff=f, n_layers=1, n_tenants=tenants, hbm_slots=tenants, n_requests=requests,
               seq_min=lo, seq_max=hi)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))
