"""The rule that gives a bf16 GEMM its kernel, swept over sizes on the CPU: every kernel gets only launches it can take."""
import numpy as np
import pytest

from tests.gemm_rule import NAMES, kernel


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
