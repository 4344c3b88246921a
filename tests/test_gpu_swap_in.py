"""Small tenants brought in while the device is idle, by kernels that read the pinned images: more of them than one launch lists, into
slots that others have lost, by a queue, sharing an image; and behind work that is still running, by the copy engine.  Which way they
came is asserted; results as of a pool where all are resident."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

D, RANK, TENANTS, SLOTS = 256, 64, 600, 300


def _brought_by_kernel(hmi, pool):
    fn = hmi.lib.hmi_internal_brought_by_kernel
    fn.restype, fn.argtypes = C.c_int64, [C.c_void_p]
    return fn(pool.h)


def _other_work():
    """Some 20 ms on the current stream."""
    big = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for _ in range(20):
        torch.mm(big, big)


def _pool(hmi, tier, block, layers, weights, shared, aliases=0):
    """aliases: that many of the last tenants have the weights of the tenants in front of them; in a host tier they share the image."""
    pool = hmi.Pool(block=block, dtype=hmi.HMI_BF16, d_model=D, d_ff=512, n_heads=D // 64, n_layers=layers, max_tenants=TENANTS,
                    hbm_slots=SLOTS if tier else TENANTS, host_tier=tier, max_requests=SLOTS, max_tokens=4 * SLOTS, ln_eps=1e-12,
                    compute_stream=torch.cuda.current_stream().cuda_stream, adapter_rank=RANK, max_classes=0)
    for layer in range(layers):
        pool.load_shared(layer, shared[layer])
    for t in range(TENANTS):
        source = t - aliases if t >= TENANTS - aliases else t
        if tier and source != t:
            pool.alias_tenant(t, source)
            continue
        for layer in range(layers):
            pool.load_tenant(t, layer, weights[(source * layers + layer) % len(weights)])
    return pool


def _weights(rng, layers):
    def bf16(*shape, scale=0.05, mean=0.0):
        return (torch.from_numpy(rng.standard_normal(shape) * scale + mean)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)

    weights = [[bf16(RANK, D, scale=0.2), bf16(RANK), bf16(D, RANK, scale=0.2), bf16(D)] for _ in range(37)]
    shared = [[bf16(3 * D, D), bf16(3 * D), bf16(D, D), bf16(D), bf16(D, mean=1.0), bf16(D), bf16(512, D), bf16(512), bf16(D, 512), bf16(D),
               bf16(D, mean=1.0), bf16(D)] for _ in range(layers)]
    return weights, shared


@pytest.mark.parametrize("layers", [2, 3])
def test_tenants_brought_in_on_an_idle_device(hmi, layers):
    rng = np.random.default_rng(layers)
    weights, shared = _weights(rng, layers)
    tiered = _pool(hmi, True, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared)
    resident = _pool(hmi, False, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared)
    try:
        before = tiered.stats()
        held = set(range(SLOTS))                 # tenants take free slots in the order in which they are loaded
        missing = 0
        for step, idle in enumerate([True, True, False, False, True]):
            ids = rng.choice(TENANTS, size=SLOTS - 1 if step != 1 else 3, replace=False).astype(np.int32)
            if step == 0:
                ids[:] = np.arange(SLOTS, 2 * SLOTS - 1)          # 299 tenants that are not there: two launches
                missing = len(set(ids.tolist()) - held)
            lens = rng.integers(1, 4, size=len(ids)).astype(np.int32)
            x = torch.from_numpy(rng.standard_normal((int(lens.sum()), D))).to(torch.bfloat16).cuda()
            y, want = torch.empty_like(x), torch.empty_like(x)
            resident.stack_forward(0, layers, x, want, ids, lens)
            brought, missed = _brought_by_kernel(hmi, tiered), tiered.stats()["misses"]
            if idle:
                torch.cuda.synchronize()
            else:
                _other_work()
            tiered.stack_forward(0, layers, x, y, ids, lens)
            assert torch.equal(y, want), step
            missed = tiered.stats()["misses"] - missed
            assert (missed > 0 or step == 1) and _brought_by_kernel(hmi, tiered) - brought == (missed if idle else 0), step
            if step == 0:
                after = tiered.stats()
                assert after["misses"] - before["misses"] == missing == SLOTS - 1
                assert after["bytes_h2d"] - before["bytes_h2d"] == missing * layers * tiered.image_bytes
    finally:
        tiered.close()
        resident.close()


@pytest.mark.parametrize("idle", [True, False])
def test_a_tenant_loaded_again_while_its_image_is_still_being_read(hmi, idle):
    """A call brings tenants in, the next one takes their slots away, and one of them is then loaded again, with nothing
    synchronised: the first call has its old weights all the same, whether a kernel (idle device) or the copy engine, which waits
    for the slots' readers behind some 20 ms of other work, has yet to read them."""
    layers, rng = 3, np.random.default_rng(5)
    weights, shared = _weights(rng, layers)
    tiered = _pool(hmi, True, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared)
    resident = _pool(hmi, False, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared)
    try:
        missing, there = np.arange(SLOTS, 2 * SLOTS, dtype=np.int32), np.arange(SLOTS, dtype=np.int32)
        again = missing[-5:]
        lens = rng.integers(1, 4, size=SLOTS).astype(np.int32)
        x = torch.from_numpy(rng.standard_normal((int(lens.sum()), D))).to(torch.bfloat16).cuda()
        old, new, y, spare, y_new = (torch.empty_like(x) for _ in range(5))
        resident.stack_forward(0, layers, x, old, missing, lens)
        torch.cuda.synchronize()
        for t in again:
            for layer in range(layers):
                resident.load_tenant(int(t), layer, weights[(int(t) * layers + layer + 11) % len(weights)])
        resident.stack_forward(0, layers, x, new, missing, lens)
        tiered.stack_forward(0, layers, x, spare, there, lens)
        torch.cuda.synchronize()
        brought = _brought_by_kernel(hmi, tiered)
        if not idle:
            _other_work()
            tiered.stack_forward(0, layers, x, spare, there, lens)
        tiered.stack_forward(0, layers, x, y, missing, lens)
        assert _brought_by_kernel(hmi, tiered) - brought == (SLOTS if idle else 0)
        tiered.stack_forward(0, layers, x, spare, there, lens)
        for t in again:
            for layer in range(layers):
                tiered.load_tenant(int(t), layer, weights[(int(t) * layers + layer + 11) % len(weights)])
        tiered.stack_forward(0, layers, x, y_new, missing, lens)
        torch.cuda.synchronize()
        assert tiered.stats()["evictions"] >= 3 * SLOTS
        assert not torch.equal(old, new)
        assert torch.equal(y, old)
        assert torch.equal(y_new, new)
    finally:
        tiered.close()
        resident.close()


def test_what_a_failed_queue_run_found_does_not_reach_the_next_call(hmi):
    """A queue's run asks whether the device is idle in front of its gather.  Where its forward is then refused (shared layers that
    nobody has loaded), the next call, behind other work, asks for itself: its tenants come by the copy engine."""
    layers, rng = 2, np.random.default_rng(7)
    weights, shared = _weights(rng, layers)
    pool = hmi.Pool(block=hmi.HMI_BLOCK_ENC_ADAPTER, dtype=hmi.HMI_BF16, d_model=D, d_ff=512, n_heads=D // 64, n_layers=layers, max_tenants=8,
                    hbm_slots=4, host_tier=True, max_requests=4, max_tokens=64, ln_eps=1e-12,
                    compute_stream=torch.cuda.current_stream().cuda_stream, adapter_rank=RANK, max_classes=0)
    queue = None
    try:
        for t in range(8):                       # the first four take the slots
            for layer in range(layers):
                pool.load_tenant(t, layer, weights[t])
        queue = hmi.Queue(pool, 4, 64, max_waiting_batches=1)
        x = torch.randn(4, D, device="cuda").to(torch.bfloat16)
        y = torch.empty_like(x)
        torch.cuda.synchronize()
        assert queue.push(0, x) is not None
        with pytest.raises(hmi.HmiError):
            queue.run()
        for layer in range(layers):
            pool.load_shared(layer, shared[layer])
        _other_work()
        pool.stack_forward(0, layers, x, y, np.arange(4, 8, dtype=np.int32), np.ones(4, dtype=np.int32))
        assert pool.stats()["misses"] == 4 and _brought_by_kernel(hmi, pool) == 0
        torch.cuda.synchronize()
        pool.stack_forward(0, layers, x, y, np.arange(4, dtype=np.int32), np.ones(4, dtype=np.int32))
        assert pool.stats()["misses"] == 8 and _brought_by_kernel(hmi, pool) == 4
        torch.cuda.synchronize()
    finally:
        if queue is not None:
            queue.close()
        pool.close()


def test_a_queue_on_an_idle_device_brings_tenants_that_share_images(hmi):
    """The first batch's tenants, all of them aliases, come by kernels (the device was idle in front of the gather of its rows), the
    next batch's by the copy engine under it."""
    layers, rng = 2, np.random.default_rng(9)
    weights, shared = _weights(rng, layers)
    tiered = _pool(hmi, True, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared, aliases=SLOTS)
    resident = _pool(hmi, False, hmi.HMI_BLOCK_ENC_ADAPTER, layers, weights, shared, aliases=SLOTS)
    queue = None
    try:
        queue = hmi.Queue(tiered, SLOTS, 4 * SLOTS, max_waiting_batches=2)
        ids = np.concatenate([rng.permutation(np.arange(SLOTS, 2 * SLOTS)), rng.permutation(SLOTS)]).astype(np.int32)
        lens = rng.integers(1, 4, size=2 * SLOTS).astype(np.int32)
        off = np.concatenate([[0], np.cumsum(lens)])
        x = torch.from_numpy(rng.standard_normal((int(off[-1]), D))).to(torch.bfloat16).cuda()
        rows = int(off[SLOTS])
        y, want = torch.empty_like(x), torch.empty_like(x)
        for first, last, at in ((0, SLOTS, slice(0, rows)), (SLOTS, 2 * SLOTS, slice(rows, None))):
            resident.stack_forward(0, layers, x[at], want[at], ids[first:last], lens[first:last])
        torch.cuda.synchronize()
        tickets = [queue.push(int(t), x[off[i]:off[i + 1]]) for i, t in enumerate(ids)]
        assert None not in tickets
        before = tiered.stats()
        for batch in range(2):
            assert queue.run() == (batch, SLOTS)
            assert _brought_by_kernel(hmi, tiered) == SLOTS
            for i in range(batch * SLOTS, (batch + 1) * SLOTS):
                queue.fetch(tickets[i], y[off[i]:off[i + 1]])
        assert torch.equal(y, want)
        assert tiered.stats()["misses"] - before["misses"] == SLOTS
        assert tiered.stats()["bytes_h2d"] - before["bytes_h2d"] == 2 * SLOTS * layers * tiered.image_bytes
    finally:
        if queue is not None:
            queue.close()
        tiered.close()
        resident.close()
