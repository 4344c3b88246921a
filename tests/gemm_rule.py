"""Which kernel the library gives a bf16 GEMM, asked of the rule itself (no GPU needed), for tests that mean a certain one."""
import ctypes as C

import numpy as np

import paper_2504_17449_amd as hmi

NAMES = ["stream", "64x64", "128x64", "128x128", "128x256", "persistent"]
COMPUTE_UNITS = 256       # of an MI355X


def kernel(ids, lens, n_out, k, gelu=False, shared=False, n_cu=COMPUTE_UNITS):
    """ids, lens: the batch's requests; shared: weights that all tenants share."""
    ids, lens = np.asarray(ids), np.asarray(lens)
    rows = [int(lens.sum())] if shared else [int(lens[ids == t].sum()) for t in np.unique(ids)]
    tiles = [sum(-(-r // m) for r in rows) for m in (256, 128)]
    fn = hmi.lib.hmi_internal_gemm_kernel
    fn.restype, fn.argtypes = C.c_int32, [C.c_int32] * 8
    return NAMES[fn(int(lens.sum()), tiles[0], tiles[1], n_out, k, int(gelu), int(shared), n_cu)]
