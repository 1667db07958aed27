"""The lookup of a cell's 8 vertex rows at the places where it can go wrong:
cells on a directory word's last bit, samples in the last cell of an axis, rows
at the end of the table, cells with inactive corners, dense and hashed levels,
every feature count, FP32, FP16 and paired tables.  Forward and adjoint against
the FP64 oracle within the FP32 rule |gpu - oracle| <= 1e-5 mag + 1e-12 (the
FP16 table is the oracle's input as rounded, so the rule is the same)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu

RES = [[64, 3, 2, 2], [65, 4, 3, 2], [130, 5, 3, 3]]  # x words of 64: full, one over, two over
RTOL, ATOL = 1e-5, 1e-12


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


def _mask():
    """A few scattered voxels, the volume's last one and one beside a word
    boundary of the second and third level among them."""
    m = np.zeros((3, 4, 6, 131), np.uint8)
    rng = np.random.default_rng(5)
    for _ in range(25):
        m[tuple(rng.integers(0, s) for s in m.shape)] = 1
    m[-1, -1, -1, -1] = 1
    m[1, 2, 3, 64] = 1
    return m


def _positions(n):
    rng = np.random.default_rng(6)
    p = rng.random((n, 4)).astype(np.float32)
    p[: n // 3, 0] = (63.0 + rng.random(n // 3)) / rng.choice([64, 129], n // 3)  # cell x = 63
    p[n // 3: n // 3 + 8] = 1.0   # the last cell of every axis
    p[n // 3 + 8: n // 3 + 16] = 0.0
    return p


def _index(fl, kind, F):
    grid = fl.grid_desc(RES, F)
    if kind == "active":
        m = _mask()
        bits = torch.from_numpy(synth.pack_mask_rows(m).view(np.int64)).cuda()
        idx, _, keep, _ = fl.fhash_build_index(grid, bits, list(m.shape[::-1]))
        return idx, O.Grid(np.array(RES), F, m), keep
    if kind == "hash":
        return fl.fhash_hash_index(grid, 8)[0], O.Grid(np.array(RES), F, hash_bits=8), None
    return fl.fhash_dense_index(grid)[0], O.Grid(np.array(RES), F), None


@pytest.mark.parametrize("table", ["f32", "f16", "paired"])
@pytest.mark.parametrize("kind", ["active", "dense", "hash"])
@pytest.mark.parametrize("F", [1, 2, 4, 8])
def test_encode_both_ways_against_oracle(fl, F, kind, table):
    idx, g, _keep = _index(fl, kind, F)
    rows, n = g.total_slots, 1021
    rng = np.random.default_rng(7)
    t = rng.uniform(-1, 1, (rows, F)).astype(np.float32)
    if table == "f16":
        t = t.astype(np.float16)
    pos = _positions(n)
    enc_ref, mag = O.encode_fwd(g, pos, t.astype(np.float64))
    dev = torch.from_numpy(t.reshape(-1)).cuda()
    if table == "paired":
        runs = torch.zeros((rows * F + 15) // 16, 2, 16, device="cuda")
        flat = torch.zeros(runs.shape[0] * 16, device="cuda")
        flat[: rows * F] = dev
        runs[:, 0] = flat.view(-1, 16)
        runs[:, 1] = float("nan")  # the gaps are never used
        dev = fl.Paired(runs.view(-1))
    p = torch.from_numpy(pos).cuda()
    enc = torch.full((n, len(RES) * F), float("nan"), device="cuda")
    fl.fhash_encode_fwd(idx, p, n, dev, enc)
    err = np.abs(enc.cpu().numpy().astype(np.float64) - enc_ref)
    assert (err <= RTOL * mag + ATOL).all(), float((err - RTOL * mag).max())
    if table != "f32":
        return
    d = rng.uniform(-1, 1, (n, len(RES) * F)).astype(np.float32)
    dt_ref, dmag = O.encode_bwd(g, pos, d.astype(np.float64))
    dt = torch.zeros(rows * F, device="cuda")
    fl.fhash_encode_bwd(idx, p, n, torch.from_numpy(d).cuda(), dt)
    err = np.abs(dt.cpu().numpy().reshape(dt_ref.shape).astype(np.float64) - dt_ref)
    assert (err <= RTOL * dmag + ATOL).all(), float((err - RTOL * dmag).max())


@pytest.mark.parametrize("F", [1, 2, 4, 8])
def test_inactive_corners_take_nothing_from_the_rows_beside_them(fl, F):
    """Rows that no active corner of the batch names may hold anything: the
    encoding is the same when they are NaN (the oracle says which those are)."""
    idx, g, _keep = _index(fl, "active", F)
    rows, n = g.total_slots, 600
    pos = _positions(n)
    used = np.zeros(rows, bool)
    slots, _ = O.corners(g, pos)
    used[np.unique(slots[slots >= 0])] = True
    used[0] = True  # corners without a row read the table's first rows, whatever they are
    rng = np.random.default_rng(8)
    t = rng.uniform(-1, 1, (rows, F)).astype(np.float32)
    bad = t.copy()
    bad[~used] = np.nan
    p = torch.from_numpy(pos).cuda()
    out = []
    for x in (t, bad):
        enc = torch.empty(n, len(RES) * F, device="cuda")
        fl.fhash_encode_fwd(idx, p, n, torch.from_numpy(x.reshape(-1)).cuda(), enc)
        out.append(enc.cpu().numpy())
    assert (~used).any()
    np.testing.assert_array_equal(out[0], out[1])
