"""Attention of a request with more blocks of queries than a grid's second index has room for: several launches, which give the bits of
one (here with few blocks a launch; the real limit is millions of rows)."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
HEADS, WIDTH = 3, 64


def _attention(hmi, qkv, lens, causal, blocks):
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    ctx = torch.full((qkv.shape[0], HEADS * WIDTH), float("nan"), device="cuda", dtype=qkv.dtype)
    fn = hmi.lib.hmi_internal_attention
    fn.restype, fn.argtypes = None, [C.c_void_p] * 3 + [C.c_int32] * 8 + [C.c_void_p]
    fn(qkv.data_ptr(), ctx.data_ptr(), off.data_ptr(), len(lens), max(lens), qkv.shape[0], HEADS * WIDTH, HEADS, int(causal),
       int(qkv.dtype == torch.bfloat16), blocks, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return ctx


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("blocks", [1, 2, 3])
def test_several_launches_are_one(hmi, dtype, causal, blocks):
    lens = [1, 700, 128, 257, 64]
    g = torch.Generator(device="cuda").manual_seed(blocks)
    qkv = torch.randn(sum(lens), 3 * HEADS * WIDTH, generator=g, device="cuda").to(dtype)
    one, several = (_attention(hmi, qkv, lens, causal, n) for n in (65535, blocks))
    assert torch.isfinite(one).all() and torch.equal(one, several)

