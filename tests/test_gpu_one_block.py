"""The one-block rounds of small volumes around the limits at which the schedule's
own rounds take over, against the oracle."""
import numpy as np
import pytest

from oracle import oracle_grow

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _instance(X, Y, Z, T, P, seed):
    """Every voxel-step admissible from 0.5, particles inside the grid whose runs of
    admissible steps are broken now and then."""
    rng = np.random.default_rng(seed)
    field = rng.uniform(0.6, 1.0, (T, Z, Y, X)).astype(np.float32)
    xyz = (rng.random((T, P, 3)) * [X, Y, Z]).astype(np.float32).clip(0, np.float32([X, Y, Z]) - np.float32(0.01))
    attr = rng.uniform(0.6, 1.0, (T, P)).astype(np.float32)
    return field, xyz, attr, np.array([[1, 2, 0, 0]], np.int32)


@pytest.mark.parametrize("schedule", ["launch", "persistent"])
@pytest.mark.parametrize("P", [191, 192, 193, 511, 512, 513])
def test_coupled_steps_around_the_limits(P, schedule):
    """16 steps a particle: 3,072 coupled steps at P = 192, 8,192 at P = 512."""
    from paper_1903_12294_amd import Grower
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    field, xyz, attr, seeds = _instance(40, 12, 9, 16, P, P)
    crit = (0.5, np.inf, 0.5, np.inf)
    ofm, opm, ost = oracle_grow(field, xyz, attr, np.array(crit, np.float32), seeds)
    assert ost["members_particle"] == 16 * P  # all of them coupled
    print(f"[one block] P={P} {schedule}", flush=True)
    with Grower(device=0, schedule=schedule) as g:
        g.load_field(field)
        g.load_particles(xyz, attr)
        g.set_criteria(*crit)
        g.set_seeds(seeds)
        for _ in range(2):
            g.grow()
            assert np.array_equal(g.read_field_mask(), ofm)
            assert np.array_equal(g.read_particle_mask(), opm)
