"""The tile depth changed in a used context (after a load that ran out of memory):
persistent rounds of the new depth, against the oracle."""
import numpy as np
import pytest

from oracle import oracle_grow
from paper_1903_12294_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("depths", [(4, 16, 8), (16, 4, 16)])
def test_depth_changes_after_a_failed_load(monkeypatch, depths):
    from paper_1903_12294_amd import Grower, _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # more candidate tiles than the one-block rounds take, at every depth
    inst = synth.make_instance(96, 48, 32, 16, 3000, n_blobs=4, seed=3, n_seeds=4, tau_f=0.01, tau_p=0.01)
    ofm, opm, _ = oracle_grow(inst["field"], inst["xyz"], inst["attr"], inst["crit"], inst["seeds"])
    g = Grower(device=0, schedule="persistent")
    try:
        for bt in depths:
            print(f"[depth] {bt}", flush=True)
            _lib.check(g.lib.mf4d_set_tile(g.ctx, bt), g.lib)
            g.load_field(inst["field"])
            g.load_particles(inst["xyz"], inst["attr"])
            g.set_criteria(*inst["crit"])
            g.set_seeds(inst["seeds"])
            g.grow()
            assert np.array_equal(g.read_field_mask(), ofm)
            assert np.array_equal(g.read_particle_mask(), opm)
            monkeypatch.setenv("MF4D_MAX_DEVICE_BYTES", "4096")
            with pytest.raises(_lib.MF4DError) as err:
                g.load_field(np.zeros((8, 40, 40, 40), np.float32))
            assert err.value.code == _lib.MF4D_ERR_OOM
            monkeypatch.delenv("MF4D_MAX_DEVICE_BYTES")
    finally:
        g.close()
