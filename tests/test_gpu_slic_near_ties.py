"""Clustering labels where two centres are as good as equally far.

The kernels fuse the products into the sums and take the hardware's square root;
the oracle rounds every operation on its own.  Labels, sums and centres of the other
tests are equal because their inputs hold no samples whose two best distances agree
that closely.  Here most point samples lie on the bisector of two centres: a label may
differ from the oracle's only there, within the bound below."""
import numpy as np
import pytest

from oracle import slic as oslic

torch = pytest.importorskip("torch")

# A distance is D = w_v |v - v_c| + w_d S.  From the same rounded differences, each
# side's D is within 7 u of the exact one (relative, u = 2^-24): the factor of time 1 u,
# so its square 2 u, the squares and their three sums 4 u, halved by the root to 3 u, the
# root 2 u (1 ulp), its product and the last sum 1 u each (the value term 2 u, so no
# more).  Two centres can rank differently only if their exact distances differ by
# less than twice that, 14 u < 2^-20.
TIE = 2.0 ** -20

K, W, CF = (2, 1, 1, 1), (1.3, 2.0, 0.0), 0.7  # no value term for the points: one centre has none


def _centres(field, xyz, attr):
    return oslic.slic(field, xyz, attr, K, W, CF, 1e-4, 0)[2]


def _case(seed, T=5, Z=9, Y=10, X=37, P=700):
    """Constant values; the field fills x >= X / 4, so that the bisector of the two seed
    cells' centres lies inside the second cell; the points are moved onto it (and the
    centres, which follow them, computed again) until both stay."""
    rng = np.random.default_rng(seed)
    field = np.full((T, Z, Y, X), 0.75, np.float32)
    field[..., :X // 4] = np.nan
    attr = np.full((T, P), 0.75, np.float32)
    xyz = (rng.random((T, P, 3)) * [1.0, Y, Z] + [0.6 * X, 0.0, 0.0]).astype(np.float32)
    t = np.broadcast_to(np.arange(T)[:, None], (T, P))
    for _ in range(30):
        c = _centres(field, xyz, attr).astype(np.float32).astype(np.float64)
        # x with equal distances from both, for each point's y, z, t
        r = [((xyz[..., 1] - c[i, 1]) ** 2 + (xyz[..., 2] - c[i, 2]) ** 2 + (CF * (t - c[i, 3])) ** 2) for i in (0, 1)]
        x = 0.5 * (c[0, 0] + c[1, 0]) + 0.5 * (r[1] - r[0]) / (c[1, 0] - c[0, 0])
        xyz[..., 0] = x.astype(np.float32)
    return field, xyz, attr


def _exact(field, xyz, c):
    """fp64 distances [points][2] from the differences as both sides round them."""
    T, P = xyz.shape[:2]
    c = c.astype(np.float32)
    p = np.concatenate([xyz.reshape(-1, 3), np.repeat(np.arange(T, dtype=np.float32), P)[:, None]], 1)
    d = (p[:, None, :] - c[None, :, :4]).astype(np.float32).astype(np.float64)
    d[..., 3] *= float(np.float32(CF))
    return float(np.float32(W[0])) * np.sqrt((d * d).sum(-1))


def test_the_inputs_hold_near_ties():
    field, xyz, attr = _case(1)
    D = _exact(field, xyz, _centres(field, xyz, attr))
    close = np.abs(D[:, 0] - D[:, 1]) < TIE * D.max(1)
    assert close.mean() > 0.5
    # and the two centres' exact distances differ there
    assert (D[close, 0] != D[close, 1]).mean() > 0.5
    # the oracle's labels there are of both kinds
    opl = oslic.slic(field, xyz, attr, K, W, CF, 1e-4, 1)[1].reshape(-1)
    assert 0.1 < opl[close].mean() < 0.9


@pytest.mark.gpu
@pytest.mark.parametrize("slabs", ["32", "31", "0"])  # boxes of samples, sample by sample, the general search
@pytest.mark.parametrize("seed", [1, 2])
def test_labels_differ_from_the_oracle_at_near_ties_only(seed, slabs, monkeypatch):
    from paper_1903_12294_amd import Grower
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("MF4D_SLIC_MASK_SLABS", slabs)
    field, xyz, attr = _case(seed)
    c0 = _centres(field, xyz, attr)
    ofl, opl, _, _, _ = oslic.slic(field, xyz, attr, K, W, CF, 1e-4, 1)
    with Grower(device=0) as g:
        g.load_field(field)
        g.load_particles(xyz, attr)
        g.slic_set_params(K, *W, CF, 1e-4, 0)
        g.slic_run()
        assert g.slic_read_centres()[0].tobytes() == c0.tobytes()
        g.slic_set_params(K, *W, CF, 1e-4, 1)
        g.slic_run()
        fl, pl = g.slic_read_labels()
    assert np.array_equal(fl, ofl)  # no field sample lies near the bisector
    D = _exact(field, xyz, c0)
    other = (pl != opl).reshape(-1)
    print(f"[near ties] {other.sum()} of {other.size} labels differ", flush=True)
    assert (np.abs(D[other, 0] - D[other, 1]) < TIE * D[other].max(1)).all()
    # away from the bisector the exact distances decide
    clear = np.abs(D[:, 0] - D[:, 1]) >= TIE * D.max(1)
    assert np.array_equal(pl.reshape(-1)[clear], D.argmin(1)[clear])
