"""The clustering's passes over boxes of samples against the search sample by
sample (MF4D_SLIC_MASK_SLABS=31 turns the boxes off) and, where it is quick, the
oracle: labels, counts and centres bit for bit, at the edges of the boxes (32 x
8 x 8 x 2 voxel-steps in blocks of 4,096, 32 x 4 x 4 x 2 below 2,048 blocks, other
shapes for planar and narrow grids), with exact ties, zero weights, samples no
window holds, lists that do not fit, and non-finite samples."""
import numpy as np
import pytest

from oracle import slic as oslic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

#        name            X    Y   Z   T   P     k               w                cf   iters  oracle
CASES = [
    ("one box",          32,  8,  8,  2,  300, (2, 2, 2, 1),    (1.0, 2.0, 2.0), 0.5, 3, True),
    ("one past a box",   33,  9,  9,  3,  301, (3, 2, 2, 2),    (1.0, 2.0, 2.0), 2.0, 3, True),
    ("single sample",    1,   1,  1,  1,  1,   (1, 1, 1, 1),    (1.0, 2.0, 2.0), 2.0, 2, True),
    ("narrow x",         7,   40, 9,  5,  63,  (1, 5, 2, 2),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("x of 16",          16,  33, 5,  4,  65,  (2, 4, 1, 2),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("planar",           45,  37, 1,  9,  500, (5, 4, 1, 3),    (1.0, 4.0, 4.0), 1.0, 4, True),
    ("planar narrow",    8,   70, 1,  17, 100, (1, 6, 1, 2),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("unvectored rows",  30,  17, 10, 4,  200, (3, 2, 2, 2),    (0.5, 4.0, 1.0), 2.0, 4, True),
    ("lists too long",   24,  16, 12, 6,  400, (12, 8, 6, 3),   (1.0, 2.0, 2.0), 1.0, 2, True),
    ("space only",       35,  15, 9,  4,  128, (5, 3, 3, 2),    (1.0, 0.0, 0.0), 1.0, 2, True),
    ("value only",       35,  15, 9,  4,  128, (5, 3, 3, 2),    (0.0, 1.0, 1.0), 1.0, 3, True),
    ("all weights zero", 35,  15, 9,  4,  128, (5, 3, 3, 2),    (0.0, 0.0, 0.0), 0.0, 2, True),
    # one term so far above the others that many distances agree to the last
    # place, where the oracle (no fused products) may rank them otherwise
    ("great weights",    35,  15, 9,  4,  128, (5, 3, 3, 2),    (1e20, 1e30, 1e25), 1e15, 2, False),
    # the sums' copies: 8, 4, 4, 2, 2, 1
    ("32 centres",       44,  18, 9,  5,  700, (4, 4, 2, 1),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("33 centres",       44,  18, 9,  5,  700, (11, 3, 1, 1),   (1.0, 4.0, 4.0), 1.0, 3, True),
    ("64 centres",       44,  18, 9,  5,  700, (4, 4, 2, 2),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("65 centres",       44,  18, 9,  5,  700, (13, 5, 1, 1),   (1.0, 4.0, 4.0), 1.0, 3, True),
    ("128 centres",      44,  18, 9,  5,  700, (8, 4, 2, 2),    (1.0, 4.0, 4.0), 1.0, 3, True),
    ("129 centres",      44,  18, 9,  5,  700, (43, 3, 1, 1),   (1.0, 4.0, 4.0), 1.0, 3, True),
    ("many blocks",      160, 96, 80, 8,  3000, (10, 6, 5, 2),  (1.0, 8.0, 8.0), 2.0, 3, False),
]


def _inputs(X, Y, Z, T, P, flat):
    rng = np.random.default_rng(X * 7 + Y * 5 + Z * 3 + T)
    field = (0.05 * rng.random((T, Z, Y, X))).astype(np.float32)
    t, z, y, x = np.meshgrid(np.arange(T), np.arange(Z), np.arange(Y), np.arange(X), indexing="ij", sparse=True)
    for _ in range(3):
        c = rng.random(4) * np.array([X, Y, Z, T])
        field += np.exp(-((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2) / 30 - (t - c[3]) ** 2 / 8).astype(np.float32)
    if flat:  # every sample of the grid alike: distances to neighbouring centres tie exactly
        field[:] = 0.25
    xyz = (rng.uniform(-0.1, 1.1, (T, P, 3)) * np.array([X, Y, Z])).astype(np.float32)
    attr = rng.random((T, P)).astype(np.float32)
    if field.size > 4:
        field.reshape(-1)[field.size // 3] = np.nan
        attr.reshape(-1)[attr.size // 2] = np.inf
        xyz[0, 0, 1] = np.nan
    return field, xyz, attr


def _run(monkeypatch, boxes, field, xyz, attr, k, w, cf, iters):
    from paper_1903_12294_amd import Grower
    monkeypatch.setenv("MF4D_SLIC_MASK_SLABS", "32" if boxes else "31")
    g = Grower(device=0)
    try:
        g.load_field(field)
        g.load_particles(xyz, attr)
        g.slic_set_params(k, *w, cf, 0.0, iters)
        it = g.slic_run()
        fl, pl = g.slic_read_labels()
        cen, cnt = g.slic_read_centres()
    finally:
        g.close()
    return it, fl, pl, cen, cnt


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_boxes_equal_sample_by_sample(monkeypatch, case, flat):
    name, X, Y, Z, T, P, k, w, cf, iters, with_oracle = case
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[slic boxes] {name} flat={flat}", flush=True)
    field, xyz, attr = _inputs(X, Y, Z, T, P, flat)
    got = _run(monkeypatch, True, field, xyz, attr, k, w, cf, iters)
    want = _run(monkeypatch, False, field, xyz, attr, k, w, cf, iters)
    for a, b in zip(got[1:], want[1:]):
        assert a.tobytes() == b.tobytes()
    assert got[0] == want[0]
    if with_oracle:
        ofl, opl, ocen, ocnt, oit = oslic.slic(field, xyz, attr, k, w, cf, 0.0, iters)
        assert got[0] == oit and np.array_equal(got[1], ofl) and np.array_equal(got[2], opl)
        assert np.array_equal(got[4], ocnt) and got[3].tobytes() == ocen.tobytes()


@pytest.mark.parametrize("k", [(8, 8, 1, 1), (13, 5, 1, 1), (16, 16, 16, 1), (17, 16, 16, 1)])
def test_merge_tiles_match_oracle(k):
    """Merging at the edges of the pair tiles (64 centres, 65, 4,096, where the
    tiles become 256 x 256, and above): features, counts, means and extents
    equal the oracle's, deviations to the 1e-9 of the other merge tests, from
    no matches to nearly all."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_12294_amd import Grower
    field, xyz, attr = _inputs(34, 32, 16, 2, 700, False)
    g = Grower(device=0)
    try:
        g.load_field(field)
        g.load_particles(xyz, attr)
        g.slic_set_params(k, 1.0, 4.0, 4.0, 1.0, 0.0, 1)
        g.slic_run()
        fl, pl = g.slic_read_labels()
        cen, cnt = g.slic_read_centres()
        for eps in (0.0, 0.01, 0.2, 5.0):
            print(f"[merge tiles] {k} eps={eps}", flush=True)
            n = g.slic_merge(eps)
            feat, st = g.slic_read_features()
            ofeat = oslic.merge_centres(cen, cnt, eps)
            assert np.array_equal(feat, ofeat) and n == int((ofeat == np.arange(len(ofeat))).sum())
            ost = oslic.feature_stats(field, xyz, attr, fl, pl, ofeat)
            exact = [0, 1, 2, 3] + list(range(6, 14))
            assert st[:, exact].tobytes() == ost[:, exact].tobytes()
            assert np.allclose(st[:, 4:6], ost[:, 4:6], rtol=1e-9, atol=1e-12)
    finally:
        g.close()
