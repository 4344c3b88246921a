"""The persistent 256 x 256 GEMM at its shortest reductions: three and four stages of 64 k (the steady state has no trip or one,
between the prologue and the hand-over to the next tile), five, and ragged segments of all sizes, short and clamped tiles among
them.  Every row compared; the dispatch is asked for the kernel, so that these sizes keep reaching it."""
import pytest

import synth
from tests.gemm_rule import kernel
from tests.test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [192, 256, 320])
def test_activation_epilogue(hmi, k):
    """First GEMM of an FFN block with few and long segments: bias and GELU, 32 column panels."""
    wl = small(synth.BLOCK_FFN, "bf16", d_model=k, d_ff=8192, n_tenants=9, hbm_slots=9, n_requests=28)
    assert kernel(*synth.batch_ids_lens(wl, 0), 8192, k, gelu=True) == "persistent"
    run_case(hmi, wl)


@pytest.mark.parametrize("k", [192, 256, 320])
def test_residual_epilogue(hmi, k):
    """Second GEMM of an FFN block: residual and fp32 result, 97 segments of 1 to some hundred rows."""
    wl = small(synth.BLOCK_FFN, "bf16", d_model=1024, d_ff=k, n_tenants=110, hbm_slots=110, n_requests=230, seq_max=110,
               popularity="uniform")
    assert kernel(*synth.batch_ids_lens(wl, 0), 1024, k) == "persistent"
    run_case(hmi, wl)


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_POSTLN, synth.BLOCK_DEC_PRELN])
def test_bias_epilogue(hmi, block):
    """QKV of a layer of d = 256."""
    wl = small(block, "bf16", d_model=256, d_ff=256, n_heads=4, n_tenants=170, hbm_slots=170, n_requests=290, seq_max=90,
               popularity="uniform")
    assert kernel(*synth.batch_ids_lens(wl, 0), 768, 256) == "persistent"
    run_case(hmi, wl)


@pytest.mark.parametrize("block", [synth.BLOCK_ENC_ADAPTER, synth.BLOCK_DEC_ADAPTER])
def test_shared_weights(hmi, block):
    """The route without tenants (rows in their own order, a last tile of 101 rows): all four GEMMs of a shared layer."""
    wl = small(block, "bf16", d_model=512, d_ff=1024, n_heads=8, n_tenants=5, hbm_slots=5, n_requests=101, seq_min=513, seq_max=513)
    ids, lens = synth.batch_ids_lens(wl, 0)
    assert int(lens.sum()) % 256 == 101
    for n_out, k in ((1536, 512), (512, 512), (1024, 512), (512, 1024)):
        assert kernel(ids, lens, n_out, k, shared=True) == "persistent", (n_out, k)
    run_case(hmi, wl, sample=[0, 1, 50, 99, 100])
