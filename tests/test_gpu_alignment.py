"""Buffers that begin off a 16-byte boundary: the same bits as from an aligned one, and nothing written beside the result."""
import pytest
import torch

import synth
from paper_2504_17449_amd import harness
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu


def shifted(t, lead):
    """A contiguous tensor of t's shape that begins `lead` elements into an allocation, and the allocation."""
    room = torch.full((t.numel() + lead + 16,), 7.0, dtype=t.dtype, device=t.device)
    return room[lead:lead + t.numel()].view(t.shape), room


@pytest.mark.parametrize("block,dtype,d,lead", [
    (synth.BLOCK_FFN, "f32", 64, 1), (synth.BLOCK_DEC_PRELN, "f32", 128, 3), (synth.BLOCK_ENC_ADAPTER, "f32", 64, 2),
    (synth.BLOCK_FFN, "bf16", 64, 2), (synth.BLOCK_ENC_POSTLN, "bf16", 256, 1),
    (synth.BLOCK_ADAPTER, "bf16", 256, 1), (synth.BLOCK_ADAPTER, "bf16", 320, 4)])   # one kernel; two GEMMs
def test_hidden_states_from_any_address(hmi, block, dtype, d, lead):
    wl = small(block, dtype, d_model=d, d_ff=64 if block == synth.BLOCK_ADAPTER else 4 * d, n_heads=d // 64, seq_max=70, n_requests=9)
    ids, lens, x = harness.batch_to_device(wl)
    pool = harness.create_pool(wl)
    try:
        harness.load_tenants(pool, wl)
        y, y_off = torch.empty_like(x), torch.empty_like(x)
        pool.forward(0, x, y, ids, lens)
        x_off, _ = shifted(x, lead)
        x_off.copy_(x)
        pool.forward(0, x_off, y_off, ids, lens)
        torch.cuda.synchronize()
    finally:
        pool.close()
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(y.view(bits), y_off.view(bits))


@pytest.mark.parametrize("max_classes", [4, 64])
def test_fp32_results_and_scores_to_any_float(hmi, max_classes):
    """The last GEMM of a pre-LN layer and the output heads write straight into the caller's buffers."""
    wl = small(synth.BLOCK_DEC_PRELN, "f32", d_model=64, d_ff=128, n_heads=1, seq_max=70, n_requests=9, max_classes=max_classes)
    ids, lens, x = harness.batch_to_device(wl)
    n = int(lens.sum())
    pool = harness.create_pool(wl)
    try:
        harness.load_tenants(pool, wl)
        y, scores, labels = torch.empty_like(x), torch.empty(n, max_classes, device=x.device), torch.empty(n, dtype=torch.int32, device=x.device)
        pool.forward(0, x, y, ids, lens)
        pool.head_forward(x, scores, labels)
        for lead in (1, 2, 3):
            y_off, y_room = shifted(y, lead)
            s_off, s_room = shifted(scores, lead)
            pool.forward(0, x, y_off, ids, lens)
            pool.head_forward(x, s_off, labels)
            torch.cuda.synchronize()
            assert torch.equal(y, y_off) and torch.equal(scores, s_off)
            for room, size in ((y_room, y.numel()), (s_room, scores.numel())):
                assert bool((room[:lead] == 7).all()) and bool((room[lead + size:] == 7).all())
    finally:
        pool.close()


@pytest.mark.parametrize("d", [256, 512, 768])
def test_static_call_from_any_address(hmi, d):
    """hmi_layer_forward_static may not allocate: such an x goes through y, and is refused where y begins elsewhere too.  Several
    units of 32 rows a workgroup, short ones among them, are adapted in place."""
    wl = small(synth.BLOCK_ADAPTER, "bf16", d_model=d, d_ff=64, n_requests=130, seq_max=200)
    ids, lens, x = harness.batch_to_device(wl)
    pool = harness.create_pool(wl)
    call = lambda a, b: hmi.hmi_layer_forward_static(pool.h, 0, a.data_ptr(), b.data_ptr(), ids, lens)
    try:
        harness.load_tenants(pool, wl)
        y, y_off = torch.empty_like(x), torch.empty_like(x)
        assert call(x, y) == hmi.HMI_OK
        for lead in (1, 4):
            x_off, _ = shifted(x, lead)
            x_off.copy_(x)
            y_off.fill_(3.0)
            assert call(x_off, y_off) == hmi.HMI_OK
            torch.cuda.synchronize()
            assert torch.equal(y.view(torch.int16), y_off.view(torch.int16)) and torch.equal(x, x_off)
            y_odd, y_room = shifted(y, 2)
            y_odd.fill_(5.0)
            assert call(x_off, y_odd) == hmi.HMI_ERR_ARG
            torch.cuda.synchronize()
            assert bool((y_odd == 5).all())
    finally:
        pool.close()
