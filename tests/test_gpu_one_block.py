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


@pytest.mark.parametrize("schedule", ["launch", "persistent"])
def test_declined_and_taken_in_turn(schedule):
    """Criteria that the one-block rounds decline (all 128 tiles admitted) and take (a
    few tiles) in turn on one context: after two declined attempts the schedule's own
    rounds are queued behind the next one.  With equal criteria, both admissibility
    modes, a round cap with resumes, a submitted grow, more than 64 seeds."""
    from paper_1903_12294_amd import Grower
    from paper_1903_12294_amd._lib import MF4D_ERR_NOT_CONVERGED, MF4DError
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X, Y, Z, T, P = 64, 64, 16, 16, 150
    field, xyz, attr, _ = _instance(X, Y, Z, T, P, 3)
    field -= 0.4                           # 0.2 .. 0.6, admitted by the wide criterion
    field[2:9, 3:12, 8:20, 30:41] += 1.0   # the narrow one's, across tiles
    attr[:, ::3] += 1.0
    seeds = np.array([[33, 9, 4, 3], [60, 60, 1, 15]], np.int32)
    many = np.concatenate([seeds, np.random.default_rng(1).integers(0, [X, Y, Z, T], (80, 4))]).astype(np.int32)
    wide, narrow = (0.1, np.inf, 0.1, np.inf), (1.1, np.inf, 1.5, np.inf)
    expect = {}

    def want(crit, sd):
        key = (crit, len(sd))
        if key not in expect:
            expect[key] = oracle_grow(field, xyz, attr, np.array(crit, np.float32), sd)
        return expect[key]

    with Grower(device=0, schedule=schedule, tile_t=4) as g:
        g.load_field(field)
        g.load_particles(xyz, attr)
        fm = torch.empty(g.field_words(), dtype=torch.int32, device="cuda:0")
        pm = torch.empty((T, P), dtype=torch.uint8, device="cuda:0")

        def check(crit, sd, how):
            print(f"[one block] {schedule} {crit[0]} {len(sd)} {how}", flush=True)
            ofm, opm, ost = want(crit, sd)
            g.set_criteria(*crit)
            g.set_seeds(sd)
            fm.fill_(-1)
            pm.fill_(9)
            torch.cuda.synchronize()
            if how == "cap":
                g.set_max_rounds(2)
                try:
                    g.grow_read(fm, pm)
                except MF4DError as e:
                    assert e.code == MF4D_ERR_NOT_CONVERGED
                    for _ in range(100):
                        try:
                            g.grow_resume()
                            break
                        except MF4DError as e:
                            assert e.code == MF4D_ERR_NOT_CONVERGED
                    g.read_field_mask(fm)
                    g.read_particle_mask(pm)
                g.set_max_rounds(0)
            elif how == "submit":
                g.grow_submit(fm, pm)
                st = g.grow_finish()
                assert st["seeds_dropped"] == ost["seeds_dropped"]
            else:
                st = g.grow_read(fm, pm)
                assert st["seeds_dropped"] == ost["seeds_dropped"]
            torch.cuda.synchronize()
            assert np.array_equal(fm.cpu().numpy().view(np.uint32), ofm)
            assert np.array_equal(pm.cpu().numpy(), opm)
            assert g.stats()["members_field"] == ost["members_field"]
            assert g.stats()["members_particle"] == ost["members_particle"]

        for crit, sd, how in [(wide, seeds, ""), (narrow, seeds, ""), (narrow, seeds, ""), (wide, seeds, ""),
                              (wide, seeds, ""), ((0.15, *wide[1:]), seeds, ""), (narrow, many, ""), (wide, many, ""),
                              ((0.15, *wide[1:]), seeds, ""), ((0.12, *wide[1:]), seeds, ""), (narrow, seeds, ""),
                              (narrow, seeds, "submit"), (wide, seeds, "submit"), ((0.12, *wide[1:]), many, "submit"),
                              ((0.15, *wide[1:]), seeds, "submit"), (narrow, seeds, "submit"),
                              (wide, seeds, "cap"), ((0.12, *wide[1:]), seeds, "cap"), (narrow, seeds, "cap"),
                              (wide, seeds, ""), ((0.15, *wide[1:]), seeds, ""), ((0.12, *wide[1:]), seeds, "cap"),
                              (narrow, seeds, "cap")]:
            check(crit, sd, how)
        g.set_admit_mode("all")
        check(narrow, seeds, "")
        g.set_admit_mode("tiles")
        check(narrow, seeds, "")
        check(wide, seeds, "")
        g.load_field(field)  # the same data again
        g.load_particles(xyz, attr)
        check(narrow, seeds, "")
