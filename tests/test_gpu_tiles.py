"""The one-workgroup-per-tile GEMM at the sizes where it can go wrong: single rows, one row past a tile, every tile size
its launch rule picks between, and (fp32) k and widths that leave half a stage or part of a tile."""
import pytest

import synth
from tests.gemm_rule import kernel
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,tenants,requests,seq,first,second", [
    (64, 64, 1, 1, 1, "stream", "stream"),             # one row, one stage of k
    (64, 192, 2, 5, 64, "64x64", "64x64"),             # whole 64-row tiles
    (128, 320, 3, 4, 65, "64x64", "64x64"),            # one row past a tile, widths that are no multiple of 128
    (768, 3072, 1, 1, 129, "64x64", "stream"),         # the long k shared by four wavefronts
    (768, 3072, 2, 9, 129, "128x64", "128x64"),        # 1 161 rows: the activation's other form sets in beyond 1 024
    (1024, 4096, 1, 3, 300, "128x128", "64x64"),       # 900 rows: 128 x 128 with the exact activation
    (1024, 2048, 8, 9, 129, "128x128", "128x64"),      # 1 161 rows of five tenants: with the polynomial
    (768, 3072, 1, 20, 133, "128x256", "128x64"),      # 2 660 rows
    (768, 3072, 1, 26, 131, "persistent", "128x128"),  # 3 406 rows: 128 x 128 with residuals, 48 stages of k
    (768, 3072, 3, 35, 131, "persistent", "128x128"),  # 4 585 rows of three tenants: its short tiles
    (768, 3072, 1, 33, 249, "persistent", "128x256"),  # 8 217 rows
    (1024, 4096, 5, 40, 150, "persistent", "128x256"), # 6 000 rows of five tenants, ragged segments
])
def test_bf16_tile_sizes(hmi, d, f, tenants, requests, seq, first, second):
    """One FFN block; first, second: the kernels that its two GEMMs are meant to get."""
    wl = small(synth.BLOCK_FFN, "bf16", d_model=d, d_ff=f, n_tenants=tenants, hbm_slots=tenants, n_requests=requests,
               seq_min=seq, seq_max=seq)
    ids, lens = synth.batch_ids_lens(wl, 0)
    assert (kernel(ids, lens, f, d, gelu=True), kernel(ids, lens, d, f)) == (first, second)
    run_case(hmi, wl, sample=sorted({0, requests // 2, requests - 1}))


@pytest.mark.parametrize("d,f,seq", [(16, 16, 1), (48, 16, 3), (16, 80, 63), (112, 64, 65), (768, 3072, 130)])
def test_fp32_tile_edges(hmi, d, f, seq):
    run_case(hmi, small(synth.BLOCK_FFN, "f32", d_model=d, d_ff=f, n_tenants=2, hbm_slots=2, n_requests=3, seq_min=1, seq_max=seq))
