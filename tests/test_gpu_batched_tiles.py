"""GPU: the batched grower in every tile shape that has a sweep of its own and in
some that share the general one (thin tiles, extents of one, where a node lies on
both faces of its tile), against the oracle: random fields (features of many
separate threads), volumes smaller than a tile and not multiples of it, few and
many words of queries."""
import numpy as np
import pytest

from tests import golden_io
from tests.test_gpu_batched import _check
from tests.test_oracle_pins import _random_instance

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4, 4, 8), (8, 4, 4, 4), (8, 8, 8, 1), (8, 8, 4, 2), (16, 4, 4, 2), (16, 8, 4, 1), (32, 4, 4, 1),
          (4, 8, 4, 4), (2, 4, 8, 8), (64, 8, 1, 1), (1, 1, 8, 64)]


@pytest.mark.parametrize("Q", [1, 33, 250])
@pytest.mark.parametrize("tile", SHAPES)
def test_tile_shapes_match_oracle(tile, Q):
    vals = np.array([0.25, 0.5, 0.75, 1.0, np.inf], np.float32)
    for seed, (X, Y, Z, T, P) in enumerate([(3, 2, 1, 2, 3), (37, 11, 9, 10, 90), (70, 9, 6, 5, 0), (17, 20, 13, 7, 30)]):
        print(f"[batched tiles] {tile} Q={Q} {X}x{Y}x{Z}x{T} P={P}", flush=True)
        rng = np.random.default_rng(31 + seed)
        inst = _random_instance(rng, X, Y, Z, T, P, 1)
        lo = rng.integers(0, 4, Q)
        crit = np.stack([vals[lo], vals[np.minimum(lo + rng.integers(0, 3, Q), 4)], vals[rng.integers(0, 3, Q)],
                         vals[rng.integers(2, 5, Q)]], 1).astype(np.float32)
        n = 6 * Q
        qseeds = np.stack([rng.integers(0, X, n), rng.integers(0, Y, n), rng.integers(0, Z, n),
                           rng.integers(0, T, n), rng.integers(0, Q, n)], 1).astype(np.int32)
        _check(inst, crit, qseeds, tile=tile)


@pytest.mark.parametrize("mode", ["both", "forward"])
@pytest.mark.parametrize("T", [16, 17, 32, 33, 64, 65, 129, 150])
def test_trajectory_lengths_match_oracle(T, mode):
    """Runs of admissible steps across the rows of 16 steps, the groups of 32 and
    64 and the pieces that a trajectory is closed in."""
    from oracle import oracle_grow_queries
    from paper_1903_12294_amd import Grower
    from tests.test_gpu_batched import _planes_to_masks, torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(T)
    X, Y, Z, P, Q = 9, 7, 5, 61, 70
    print(f"[batched tiles] T={T} {mode}", flush=True)
    inst = _random_instance(rng, X, Y, Z, T, P, 1)
    inst["attr"] = np.where(rng.random((T, P)) < 0.97, np.float32(1.0), inst["attr"]).astype(np.float32)
    vals = np.array([0.25, 0.5, 1.0, np.inf], np.float32)
    lo = rng.integers(0, 3, Q)
    crit = np.stack([vals[lo], vals[np.minimum(lo + 1, 3)], vals[rng.integers(0, 3, Q)],
                     np.full(Q, np.inf, np.float32)], 1).astype(np.float32)
    n = 4 * Q
    qseeds = np.stack([rng.integers(0, X, n), rng.integers(0, Y, n), rng.integers(0, Z, n),
                       rng.integers(0, T, n), rng.integers(0, Q, n)], 1).astype(np.int32)
    with Grower(device=0) as g:
        g.set_trajectory_mode(mode)
        g.load_field(inst["field"])
        g.load_particles(inst["xyz"], inst["attr"])
        g.set_queries(crit, qseeds)
        fp, pp, _ = g.grow_batched()
    res = oracle_grow_queries(inst["field"], inst["xyz"], inst["attr"], crit, qseeds, forward_only=mode == "forward")
    assert any(r[1].sum() > 2 * T for r in res.values())
    for q, (ofm, opm, _) in res.items():
        f, p = _planes_to_masks(fp, pp, inst["field"].shape, T, P, q)
        assert np.array_equal(f, golden_io.unpack_field(ofm, inst["field"].shape)), q
        assert np.array_equal(p, opm), q
