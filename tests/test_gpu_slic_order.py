"""Clustering of few long trajectories: the order of the point samples is built in
chunks of 64 particles x 64 steps (both remainders, one particle, the edges of a
chunk), against the oracle."""
import numpy as np
import pytest

from oracle import slic as oslic

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("P,Tp", [(1, 64), (1, 200), (63, 65), (64, 128), (65, 129), (130, 63)])
def test_long_trajectories_match_oracle(P, Tp):
    from paper_1903_12294_amd import Grower
    from tests.test_gpu_slic import _case
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rate = 20
    T, Z, Y, X = 10, 6, 7, 12
    field, _, _ = _case(3, T, Z, Y, X, 0)
    _, xyz, attr = _case(4 + P, Tp, Z, Y, X, P, spread=1.2)
    k, w, cf, eps, it = (3, 2, 2, 2), (1.0, 2.0, 2.0), 0.5, 1e-4, 5
    print(f"[order] P={P} Tp={Tp}", flush=True)
    with Grower(device=0) as g:
        g.load_field(field)
        g.load_particles(xyz, attr, rate=rate)
        g.slic_set_params(k, w[0], w[1], w[2], cf, eps, it)
        n_it = g.slic_run()
        fl, pl = g.slic_read_labels()
        cen, cnt = g.slic_read_centres()
    ofl, opl, ocen, ocnt, oit = oslic.slic(field, xyz, attr, k, w, cf, eps, it, rate=rate)
    assert n_it == oit
    assert np.array_equal(fl, ofl) and np.array_equal(pl, opl)
    assert np.array_equal(cnt, ocnt) and cen.tobytes() == ocen.tobytes()
