"""Calls captured into a graph: at any point of a pool's life, replayed after other calls with other batches, with the eager
call's bits every time."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_17449_amd import harness
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu


def check(wl, forward, before, between, **pool_kw):
    """Captures forward(pool, x, y, ids, lens) after `before` calls outside a graph; three replays, `between` calls on another
    batch in front of each."""
    side = torch.cuda.Stream()
    batches = [harness.batch_to_device(wl, b) for b in range(2)]
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        pool = harness.create_pool(wl, max_tokens=max(int(lens.sum()) for _, lens, _ in batches), **pool_kw)
        try:
            harness.load_tenants(pool, wl)
            want = [torch.empty_like(x) for _, _, x in batches]
            for _ in range(before):
                for (ids, lens, x), y in zip(batches, want):
                    forward(pool, x, y, ids, lens)
            ids, lens, x = batches[0]
            y = torch.empty_like(x)
            graph = torch.cuda.CUDAGraph()
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                forward(pool, x, y, ids, lens)
            other = torch.empty_like(batches[1][2])
            for _ in range(3):
                for _ in range(between):
                    forward(pool, batches[1][2], other, batches[1][0], batches[1][1])
                y.fill_(3.0)
                graph.replay()
                forward(pool, batches[1][2], other, batches[1][0], batches[1][1])
                side.synchronize()
                assert torch.equal(y.view(torch.int16), want[0].view(torch.int16))
                assert torch.equal(other.view(torch.int16), want[1].view(torch.int16))
        finally:
            side.synchronize()
            pool.close()


@pytest.mark.parametrize("before", [1, 3, 4, 8, 12])          # twice as many calls: the ring of index buffers has 16, in two marks
def test_static_call_captured(hmi, before):
    def forward(pool, x, y, ids, lens):
        assert hmi.hmi_layer_forward_static(pool.h, 0, x.data_ptr(), y.data_ptr(), ids, lens) == hmi.HMI_OK, hmi.hmi_last_error(pool.h)
    check(small(synth.BLOCK_ADAPTER, "bf16", d_model=256, d_ff=64, n_requests=40, seq_max=60), forward, before, 20)


def test_forward_of_300_requests_captured(hmi):
    """More index values than the arguments of one kernel hold."""
    check(small(synth.BLOCK_FFN, "bf16", d_model=256, d_ff=256, n_requests=300, seq_max=9), lambda pool, *a: pool.forward(0, *a), 8, 20)
