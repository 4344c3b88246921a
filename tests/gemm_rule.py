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


FORMS = ["one line", "32x32", "32x64", "64x64", "128x64"]       # of k a stage; the others take two
FORMS_F32 = ["32x32", "64x32", "64x64"]


def _rows(ids, lens, shared):
    ids, lens = np.asarray(ids), np.asarray(lens)
    return [int(lens.sum())] if shared else [int(lens[ids == t].sum()) for t in np.unique(ids)]


def form(ids, lens, n_out, k, gelu=False, shared=False, n_cu=COMPUTE_UNITS):
    """Which tile kernel a bf16 launch gets whose `kernel` is 64x64 or 128x64."""
    rows = _rows(ids, lens, shared)
    tiles = [sum(-(-r // m) for r in rows) for m in (256, 128)]
    fn = hmi.lib.hmi_internal_gemm_form
    fn.restype, fn.argtypes = C.c_int32, [C.c_int32] * 8
    return FORMS[fn(sum(rows), tiles[0], tiles[1], n_out, k, int(gelu), int(shared), n_cu)]


def form_f32(ids, lens, n_out, k, shared=False, n_cu=COMPUTE_UNITS):
    """Which tile kernel an fp32 launch gets."""
    rows = _rows(ids, lens, shared)
    fn = hmi.lib.hmi_internal_gemm_form_f32
    fn.restype, fn.argtypes = C.c_int32, [C.c_int32] * 6
    return FORMS_F32[fn(sum(rows), sum(-(-r // 64) for r in rows), n_out, k, int(shared), n_cu)]


def adapter_unit(rows, with_norm, n_cu=COMPUTE_UNITS):
    """Rows of a unit of the adapter kernel (0: the general form) for a batch of rows[i] rows of its i-th tenant."""
    units = [sum(-(-int(r) // n) for r in rows) for n in (8, 16, 32)]
    fn = hmi.lib.hmi_internal_adapter_unit
    fn.restype, fn.argtypes = C.c_int32, [C.c_int32] * 6
    return fn(len(rows), *units, int(with_norm), n_cu)
