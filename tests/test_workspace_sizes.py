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


def _index_query(res, dims, layout):
    m, nb = fl.MaskDesc(), C.c_size_t(0)
    m.bits = 1 << 20
    for d in range(4):
        m.dims[d] = dims[d]
    rc = fl.lib().fhash_build_index(C.byref(fl.grid_desc(res, 2, layout)), C.byref(m), None, None,
                                    C.byref(nb), None, None, None)
    assert rc == fl.OK, fl.lib().fhash_last_error()
    return nb.value


def _axis_passes(res, dims, layout):
    """Bytes of a build that reduces the mask along t, z and y in turn between two
    arrays and then has the directory beside them, each as large as the level that
    needs most of it."""
    Sx, Sy, Sz, T = dims
    W = (Sx + 63) // 64
    top = [0, 0, 0, 0]
    for x, y, z, t in res:
        wc, wv = (x + 62) // 64, (x + 63) // 64
        bricks = ((t + 1) // 2) * ((z + 1) // 2) * ((y + 1) // 2) * (((x + 1) // 2 + 3) // 4)
        use = [max((t - 1) * Sz * Sy * W, (t - 1) * (z - 1) * (y - 1) * W,
                   t * (z - 1) * (y - 1) * wc, t * z * y * wc),
               max((t - 1) * (z - 1) * Sy * W, (t - 1) * (z - 1) * (y - 1) * wc,
                   t * z * (y - 1) * wc),
               2 * t * z * y * wv, 2 * bricks if layout else 0]
        top = [max(a, b) for a, b in zip(top, use)]
    return 8 * sum(top)


@pytest.mark.parametrize("layout", [0, 1])
def test_index_workspace_stays_within_a_pass_per_axis(layout):
    """Above 256 MB the build asks for no more than that, whatever the levels."""
    rng = np.random.default_rng(layout)
    large = 0
    for _ in range(400):
        dims = [int(v) for v in np.exp(rng.uniform(np.log([100, 100, 40, 10]),
                                                   np.log([1500, 1500, 600, 200])))]
        fine = rng.uniform(0.1, 1.0)
        L = int(rng.integers(1, 17))
        res = [[max(2, int(S * fine ** (k > 0) * rng.uniform(0.6, 1.0) ** (L - 1 - l)))
                for k, S in enumerate(dims)] for l in range(L)]
        need, most = _index_query(res, dims, layout), _axis_passes(res, dims, layout)
        assert need <= max(most, 256 << 20) + (1 << 16), (dims, res, need, most)
        large += most > 256 << 20
    assert large > 50
