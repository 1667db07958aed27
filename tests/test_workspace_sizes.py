"""The workspace queries of the fused backward calls (host only): the size never
falls as the batch grows, so a workspace sized once for the largest batch is
accepted for every smaller one."""
import ctypes as C

import numpy as np
import pytest

from paper_2507_03836_amd import _lib as fl

FAKE = C.c_void_p(1 << 20)  # aligned, never dereferenced: the query ends first
FOLD = [[2, 2, 2, 2], [4, 6, 2, 2], [8, 12, 2, 2], [15, 23, 4, 2], [30, 45, 8, 3], [60, 90, 15, 5]]


def _query(call, idx, mlp, n, flags):
    L, nb = fl.lib(), C.c_size_t(0)
    head = (C.byref(idx), C.byref(mlp), FAKE)
    if call == "bwd":
        rc = L.fhash_fused_bwd(*head, C.c_int64(n), FAKE, fl.F32, FAKE, None, FAKE, FAKE, FAKE,
                               C.c_uint32(flags), None, None, C.byref(nb), None)
    else:
        rc = L.fhash_fused_train(*head, FAKE, C.c_int64(n), FAKE, fl.F32, FAKE, None,
                                 C.c_float(1.0), FAKE, FAKE, None, C.c_uint32(flags), None, None,
                                 C.byref(nb), None)
    assert rc == fl.OK, L.fhash_last_error()
    return nb.value


@pytest.mark.parametrize("flags", [0, fl.SAMPLES_SORTED, fl.COARSE_LDS])
@pytest.mark.parametrize("kind,F,hidden", [("dense", 2, [64, 64, 64]), ("dense", 1, [32]),
                                           ("dense", 4, [64, 64]), ("hash", 2, [64, 64])])
@pytest.mark.parametrize("call", ["bwd", "train"])
def test_size_never_falls_with_the_batch(call, kind, F, hidden, flags):
    grid = fl.grid_desc(FOLD, F)
    idx = (fl.fhash_hash_index(grid, 9) if kind == "hash" else fl.fhash_dense_index(grid))[0]
    mlp = fl.mlp_desc([len(FOLD) * F] + hidden + [1])
    at = sorted({1, *range(1, 40001, 16), *range(0, 40001, 2048), *range(1, 40001, 2048)}
                | {int(x) for x in np.logspace(4.7, 7.3, 200)})
    size = [_query(call, idx, mlp, n, flags) for n in at]
    fall = [(a, b, x, y) for a, b, x, y in zip(at, at[1:], size, size[1:]) if y < x]
    assert not fall, fall[:3]
