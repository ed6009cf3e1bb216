"""GPU: grows at the sizes where the launches change form, against the oracle:
rows that are not whole 16-byte vectors or 32-bit words, particle counts around
16 and outputs off a 16-byte boundary, up to and over 64 seeds, volumes on both
sides of the one-block rounds' limits (tiles of the volume, candidate tiles,
coupled steps) and of the shared admissibility launch's (8,192 tiles), each
grown twice and with its read-outs queued."""
import numpy as np
import pytest

from oracle import oracle_grow
from paper_1903_12294_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# X, Y, Z, T, P, seeds, tile depth, criterion low
SHAPES = [
    (1, 1, 1, 1, 0, 1, 4, -9.0),
    (5, 9, 7, 3, 1, 2, 4, 0.2),
    (33, 17, 9, 5, 15, 63, 8, 0.2),
    (36, 8, 11, 17, 16, 64, 16, 0.2),
    (63, 10, 8, 9, 17, 65, 4, 0.2),
    (128, 9, 8, 6, 48, 3, 4, 0.2),
    (64, 64, 64, 4, 33, 2, 4, -9.0),       # 128 candidate tiles: the block declines
    (64, 64, 64, 16, 40, 70, 4, 0.3),      # 512 tiles in all
    (65, 64, 64, 16, 40, 4, 4, 0.3),       # more than 512
    (32, 32, 16, 24, 700, 2, 8, -9.0),     # more than 8,192 coupled steps
    (3, 128, 128, 132, 20, 3, 4, -9.0),    # more than 8,192 tiles
]


@pytest.mark.parametrize("device_seeds", [False, True])
@pytest.mark.parametrize("X,Y,Z,T,P,S,bt,lo", SHAPES)
def test_edges_match_oracle(X, Y, Z, T, P, S, bt, lo, device_seeds):
    from paper_1903_12294_amd import Grower
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[grow edges] {X}x{Y}x{Z}x{T} P={P} S={S} bt={bt} lo={lo} device={device_seeds}", flush=True)
    rng = np.random.default_rng(X * 1000 + T)
    i = synth.make_instance(X, Y, Z, T, P, n_blobs=4, seed=5, n_seeds=1)
    crit = np.array([lo, np.inf, lo, np.inf], np.float32)
    seeds = np.concatenate([i["seeds"].reshape(-1, 4)[:1],
                            rng.integers(0, [X, Y, Z, T], (S - 1, 4))]).astype(np.int32)
    xyz = i["xyz"] if P else np.zeros((T, 0, 3), np.float32)
    attr = i["attr"] if P else np.zeros((T, 0), np.float32)
    ofm, opm, ost = oracle_grow(i["field"], xyz, attr, crit, seeds)
    dev = torch.device("cuda:0")
    with Grower(device=0, tile_t=bt) as g:
        g.load_field(i["field"])
        if P:
            g.load_particles(i["xyz"], i["attr"])
        g.set_criteria(*crit)
        g.set_seeds(torch.from_numpy(seeds).to(dev) if device_seeds else seeds)
        for off in (0, 1, 3):
            fm = torch.full((g.field_words() + off,), -1, dtype=torch.int32, device=dev)
            pm = torch.full((T * P + off,), 0xFF, dtype=torch.uint8, device=dev)
            torch.cuda.synchronize()
            g.grow_read(fm[off:], pm[off:] if P else None)
            torch.cuda.synchronize()
            assert np.array_equal(fm[off:].cpu().numpy().view(np.uint32), ofm), off
            assert np.array_equal(pm[off:].cpu().numpy(), opm.reshape(-1)), off
            assert (fm[:off].cpu() == -1).all() and (pm[:off].cpu() == 0xFF).all()
            st = g.stats()
            assert st["members_field"] == ost["members_field"]
            assert st["members_particle"] == ost["members_particle"]
            g.grow()
            assert np.array_equal(g.read_field_mask(), ofm)
            if P:
                assert np.array_equal(g.read_particle_mask(), opm)


@pytest.mark.parametrize("mode", ["both", "forward"])
@pytest.mark.parametrize("schedule", ["launch", "persistent"])
@pytest.mark.parametrize("T,P", [(65, 90), (128, 64), (129, 33), (192, 200), (200, 1), (256, 65), (257, 70)])
def test_long_trajectories_match_oracle(T, P, schedule, mode):
    """Two to five label words a trajectory, with runs of admissible steps across
    their boundaries."""
    from paper_1903_12294_amd import Grower
    from tests.test_oracle_pins import _random_instance
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[grow edges] T={T} P={P} {schedule} {mode}", flush=True)
    rng = np.random.default_rng(T + P)
    i = _random_instance(rng, 11, 6, 5, T, P, 6)
    i["attr"] = np.where(rng.random((T, P)) < 0.98, np.float32(1.0), i["attr"]).astype(np.float32)
    crit = np.array([0.75, np.inf, 0.75, np.inf], np.float32)
    ofm, opm, ost = oracle_grow(i["field"], i["xyz"], i["attr"], crit, i["seeds"], forward_only=mode == "forward")
    assert ost["members_particle"] > T // 2
    with Grower(device=0, schedule=schedule) as g:
        g.set_trajectory_mode(mode)
        g.load_field(i["field"])
        g.load_particles(i["xyz"], i["attr"])
        g.set_criteria(*crit)
        g.set_seeds(i["seeds"])
        for _ in range(2):
            g.grow()
            assert np.array_equal(g.read_field_mask(), ofm)
            assert np.array_equal(g.read_particle_mask(), opm)


@pytest.mark.parametrize("P", [31, 32, 33, 8191, 8193, 16385, 300000])
def test_admission_chunks_match_oracle(P):
    """Particle counts around the sizes at which a block's share of the admission
    doubles."""
    from paper_1903_12294_amd import Grower
    from tests.test_oracle_pins import _random_instance
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[grow edges] admission P={P}", flush=True)
    i = _random_instance(np.random.default_rng(P), 16, 9, 7, 5, P, 4)
    crit = np.array([0.5, np.inf, 0.75, np.inf], np.float32)
    ofm, opm, ost = oracle_grow(i["field"], i["xyz"], i["attr"], crit, i["seeds"])
    assert ost["members_particle"] > P // 10
    with Grower(device=0) as g:
        g.load_field(i["field"])
        g.load_particles(i["xyz"], i["attr"])
        g.set_criteria(*crit)
        g.set_seeds(i["seeds"])
        g.grow()
        assert np.array_equal(g.read_field_mask(), ofm)
        assert np.array_equal(g.read_particle_mask(), opm)
