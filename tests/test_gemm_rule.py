"""The rules that give a GEMM and the adapter their kernels, swept over sizes on the CPU: every kernel gets only launches it can take,
and the GPU tests that mean certain forms reach them."""
import itertools

import numpy as np
import pytest

import synth
from tests.gemm_rule import FORMS, FORMS_F32, NAMES, adapter_unit, form, form_f32, kernel


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_cu", [256, 64, 32])
def test_every_launch_gets_a_kernel_that_takes_it(shared, n_cu):
    rng = np.random.default_rng(n_cu + shared)
    seen = set()
    for _ in range(4000):
        n_out = 64 * int(rng.integers(1, 97))
        k = 64 * int(rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 48, 64]))
        tenants = int(np.exp(rng.uniform(0, np.log(300))))
        lens = np.maximum(1, np.exp(rng.uniform(0, np.log(6000 / tenants + 2), tenants)).astype(int))
        name = kernel(np.arange(tenants), lens, n_out, k, bool(rng.integers(0, 2)), shared, n_cu)
        seen.add(name)
        rows, per_tile = int(lens.sum()), sum(-(-int(n) // 128) for n in ([lens.sum()] if shared else lens))
        if name == "persistent":
            assert n_out % 256 == 0 and k >= 192
        if name == "128x256":
            assert n_out % 256 == 0
        if name == "128x128":
            assert n_out % 128 == 0
        if name == "stream":
            # whole columns of 32; all tenants' rows few, or k shared by four wavefronts, one workgroup an item
            assert n_out % 32 == 0
            assert (not shared and rows <= 32 * per_tile) or (k % 256 == 0 and k >= 1536 and -(-rows // 32) * (n_out // 32) <= n_cu)
    assert seen == set(NAMES)


def _batch(rng, tokens):
    tenants = int(np.exp(rng.uniform(0, np.log(300))))
    return np.arange(tenants), np.maximum(1, np.exp(rng.uniform(0, np.log(tokens / tenants + 2), tenants)).astype(int))


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_cu", [256, 64])
def test_forms_with_two_lines_of_k_are_one_round(shared, n_cu):
    rng = np.random.default_rng(n_cu + shared)
    heights = {"32x32": (32, 32), "32x64": (32, 64), "64x64": (64, 64), "128x64": (128, 64)}
    seen = set()
    for _ in range(4000):
        n_out, k = 64 * int(rng.integers(1, 97)), 64 * int(rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 48, 64]))
        ids, lens = _batch(rng, 3000)
        gelu = bool(rng.integers(0, 2))
        name, tile = kernel(ids, lens, n_out, k, gelu, shared, n_cu), form(ids, lens, n_out, k, gelu, shared, n_cu)
        seen.add(tile)
        if tile == "one line":
            continue
        bm, bn = heights[tile]
        assert name == ("128x64" if bm == 128 else "64x64") and k % 128 == 0
        # an entry of a tenant's list of 128-row tiles counts with all the tiles it has room for
        m_tiles = -(-int(lens.sum()) // bm) if shared else sum(-(-int(n) // 128) for n in lens) * (128 // bm)
        assert m_tiles * -(-n_out // bn) <= n_cu
    assert seen == set(FORMS)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_cu", [256, 64])
def test_fp32_forms_take_their_launches(shared, n_cu):
    rng = np.random.default_rng(n_cu + shared)
    seen = set()
    for _ in range(4000):
        n_out, k = 16 * int(rng.integers(1, 200)), 16 * int(rng.integers(1, 100))
        ids, lens = _batch(rng, 3000)
        tile = form_f32(ids, lens, n_out, k, shared, n_cu)
        seen.add(tile)
        assert k % {"32x32": 128, "64x32": 64, "64x64": 16}[tile] == 0
        if tile == "32x32":
            assert (-(-int(lens.sum()) // 32) if shared else sum(-(-int(n) // 64) for n in lens) * 2) * -(-n_out // 32) <= n_cu
    assert seen == set(FORMS_F32)


@pytest.mark.parametrize("with_norm", [False, True])
@pytest.mark.parametrize("n_cu", [256, 64])
def test_adapter_units_are_a_workgroup_each(with_norm, n_cu):
    rng = np.random.default_rng(n_cu + with_norm)
    seen = set()
    for _ in range(4000):
        _, rows = _batch(rng, 20000)
        unit = adapter_unit(rows, with_norm, n_cu)
        seen.add(unit)
        if unit:
            assert len(rows) <= 256 and sum(-(-int(r) // unit) for r in rows) <= n_cu
    assert seen == ({0, 8, 16, 32} if with_norm else {0, 8, 32})


def _cases(fn):
    """The parametrised cases of a test, as dicts."""
    sets = []
    for mark in fn.pytestmark:
        if mark.name == "parametrize":
            names = mark.args[0].split(",")
            sets.append([dict(zip(names, v if len(names) > 1 else (v,))) for v in mark.args[1]])
    for parts in itertools.product(*sets):
        yield {k: v for part in parts for k, v in part.items()}


def test_the_gpu_tests_of_small_launches_reach_every_form():
    """tests/test_gpu_small_launches.py names sizes and means forms."""
    from tests import test_gpu_small_launches as T
    from tests.test_gpu_parity import small

    def launches(c, dtype, tenants, block):
        d, f = c["d"], c["f"]
        wl = small(block, dtype, d_model=d, d_ff=f, n_heads=d // 64, n_tenants=tenants, hbm_slots=tenants, n_requests=c["requests"],
                   seq_min=c["lo"], seq_max=c["hi"])
        ids, lens = synth.batch_ids_lens(wl)
        for n_out, k, gelu in [(f, d, True), (d, f, False)] + ([(3 * d, d, False), (d, d, False)] if block != synth.BLOCK_FFN else []):
            yield ids, lens, n_out, k, gelu

    for fn, shared in ((T.test_shared_weights, True), (T.test_a_tenants_own_weights, False)):
        seen = set()
        for c in _cases(fn):
            for ids, lens, n_out, k, gelu in launches(c, "bf16", c.get("tenants", 3), c["block"]):
                name = kernel(ids, lens, n_out, k, gelu, shared)
                seen.add(form(ids, lens, n_out, k, gelu, shared) if name in ("64x64", "128x64") else name)
        assert seen >= set(FORMS) | {"stream"}, fn.__name__
    seen = set()
    for c in _cases(T.test_fp32_tiles):
        for ids, lens, n_out, k, _ in launches(c, "f32", c["tenants"], synth.BLOCK_FFN):
            seen.add(form_f32(ids, lens, n_out, k))
    assert seen == set(FORMS_F32)
