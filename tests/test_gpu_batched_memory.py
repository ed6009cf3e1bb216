"""What a batched grow holds beside the caller's planes: four bytes of ranks for each
voxel-step and particle-step, and the tiles' lists."""
import numpy as np
import pytest

from paper_1903_12294_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rate", [1, 3])
def test_scratch_of_a_batched_grow(rate):
    from paper_1903_12294_amd import Grower, _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    X, Y, Z, T, P = 48, 40, 16, 10, 60000
    i = synth.make_instance(X, Y, Z, T, P, n_blobs=4, seed=2, n_seeds=2, tau_f=0.25, tau_p=0.25, rate=rate)
    V, Tp = X * Y * Z * T, T * rate
    Tpad = 1 << (Tp - 1).bit_length()
    lib = _lib.load_library()
    with Grower(device=0) as g:
        g.set_batched_tile(8, 4, 4, 4)
        g.load_field(i["field"])
        g.load_particles(i["xyz"], i["attr"], rate=rate)
        crit = np.array([[0.2, np.inf, 0.2, np.inf]] * 5, np.float32)
        seeds = np.concatenate([np.tile(i["seeds"][:1], (5, 1)), np.arange(5)[:, None]], 1).astype(np.int32)
        g.set_queries(crit, seeds)
        f = torch.empty((V, 8), dtype=torch.int32, device="cuda:0")
        p = torch.empty((Tp, P, 8), dtype=torch.int32, device="cuda:0")
        held = lib.mf4d_device_bytes()
        g.grow_batched(f, p)
        ntb = -(-X // 8) * -(-Y // 4) * -(-Z // 4) * -(-T // 4)
        # a tile: flags 8, steps 8, lists 16 bytes rounded up to 64 sub-lists, activity 1
        lists = 64 * 1024 + 2 * 64 * 8 + 64 * 128 * 3
        assert lib.mf4d_device_bytes() - held <= 4 * V + 4 * P * Tpad + 33 * ntb + lists
