"""The particle read-out around the sizes at which a thread's share of the steps
changes (16, 32, 64 and more) and the remainders of its 16 particles, queued behind a
grow and on its own, aligned and not, against the oracle."""
import numpy as np
import pytest

from oracle import oracle_grow

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("P,T", [(1, 15), (15, 16), (16, 17), (17, 33), (4095, 31), (4097, 32), (999, 130), (33, 64),
                                 (70000, 20), (2097152, 3), (2097153, 3)])
def test_shares_match_oracle(P, T):
    from paper_1903_12294_amd import Grower
    from tests.test_oracle_pins import _random_instance
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[particle read] P={P} T={T}", flush=True)
    i = _random_instance(np.random.default_rng(P + T), 9, 7, 5, T, P, 4)
    crit = np.array([0.5, np.inf, 0.75, np.inf], np.float32)
    _, opm, ost = oracle_grow(i["field"], i["xyz"], i["attr"], crit, i["seeds"])
    with Grower(device=0) as g:
        g.load_field(i["field"])
        g.load_particles(i["xyz"], i["attr"])
        g.set_criteria(*crit)
        g.set_seeds(i["seeds"])
        for off in (0, 1):
            out = torch.full((T * P + off + 16,), 7, dtype=torch.uint8, device="cuda:0")
            for queued in (True, False):
                out.fill_(7)
                torch.cuda.synchronize()
                if queued:
                    g.grow_read(None, out[off:off + T * P])
                else:
                    g.read_particle_mask(out[off:off + T * P])
                torch.cuda.synchronize()
                assert np.array_equal(out[off:off + T * P].cpu().numpy(), opm.reshape(-1))
                assert (out[:off] == 7).all() and (out[off + T * P:] == 7).all()
                assert g.stats()["members_particle"] == ost["members_particle"]
