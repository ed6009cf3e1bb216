"""Loading again into one context: buffers of a load of the same sizes are kept,
every result is that of a fresh context, and what is kept is given back."""
import numpy as np
import pytest

from oracle import oracle_grow
from paper_1903_12294_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _inst(seed, X=37, Y=19, Z=11, T=9, P=201, rate=1):
    i = synth.make_instance(X, Y, Z, T, P, n_blobs=4, seed=seed, n_seeds=4, tau_f=0.25, tau_p=0.25, rate=rate)
    i["field"].reshape(-1)[seed] = np.nan
    if P:
        i["attr"].reshape(-1)[seed] = np.nan
    return i


def _load(g, i, device):
    put = (lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")) if device else np.ascontiguousarray
    g.load_field(put(i["field"]))
    if i["P"]:
        g.load_particles(put(i["xyz"]), put(i["attr"]), rate=i["rate"])


def _check(g, i):
    g.set_criteria(*i["crit"])
    g.set_seeds(i["seeds"])
    g.grow()
    fm = g.read_field_mask()
    pm = g.read_particle_mask() if i["P"] else None
    xyz = i["xyz"] if i["P"] else np.zeros((i["T"], 0, 3), np.float32)
    attr = i["attr"] if i["P"] else np.zeros((i["T"], 0), np.float32)
    ofm, opm, _ = oracle_grow(i["field"], xyz, attr, i["crit"], i["seeds"], rate=i["rate"])
    assert np.array_equal(fm, ofm)
    if i["P"]:
        assert np.array_equal(pm, opm)


@pytest.mark.parametrize("device", [True, False])
def test_reloads_match_oracle(device):
    """Same sizes again and again (both kinds of buffer kept), other particles
    on the same field sizes, no particles, another rate, another field size,
    with asynchronous read-outs and a clustering in between."""
    from paper_1903_12294_amd import Grower, _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = _lib.load_library()
    before = lib.mf4d_device_bytes()
    g = Grower(device=0)
    try:
        seq = [_inst(1), _inst(2), _inst(3, P=70), _inst(4, P=70), _inst(5, P=0), _inst(6), _inst(7, rate=3),
               _inst(8, rate=3), _inst(9, X=40), _inst(10, X=40)]
        for n, i in enumerate(seq):
            print(f"[reload] {n}", flush=True)
            _load(g, i, device)
            _check(g, i)
            if n in (1, 6):  # label sets swapped, clustering buffers made
                g.set_read_async(True)
                f = torch.empty(g.field_words(), dtype=torch.int32, device="cuda:0")
                for _ in range(3):
                    g.grow_read(f, None)
                g.set_read_async(False)
                g.slic_set_params((3, 2, 2, 2), 1.0, 2.0, 2.0, 1.0, 0.0, 2)
                g.slic_run()
    finally:
        g.close()
    assert lib.mf4d_device_bytes() == before


def test_kept_buffers_are_given_back():
    """After a field load the particle buffers of the load before stay for the
    particles expected next; a grow without them gives them back."""
    from paper_1903_12294_amd import Grower, _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = _lib.load_library()
    i = _inst(1)
    g = Grower(device=0)
    try:
        g.load_field(i["field"])
        alone = lib.mf4d_device_bytes()
        g.load_particles(i["xyz"], i["attr"])
        both = lib.mf4d_device_bytes()
        g.load_field(i["field"])
        g.load_particles(i["xyz"], i["attr"])
        assert lib.mf4d_device_bytes() == both
        g.load_field(i["field"])
        assert lib.mf4d_device_bytes() == both
        g.set_criteria(*i["crit"])
        g.set_seeds(i["seeds"])
        g.grow()
        assert lib.mf4d_device_bytes() == alone  # (a few seeds need no buffer)
        with pytest.raises(_lib.MF4DError):
            g.read_particle_mask(np.zeros((i["T"], i["P"]), np.uint8))
    finally:
        g.close()


def test_unaligned_device_field():
    """A device field that starts 4 bytes past a 16-byte boundary."""
    from paper_1903_12294_amd import Grower
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    i = _inst(3, X=36, P=50)
    n = i["field"].size
    buf = torch.empty(n + 1, dtype=torch.float32, device="cuda:0")
    buf[1:] = torch.from_numpy(i["field"].reshape(-1))
    g = Grower(device=0)
    try:
        g.load_field(buf[1:].view(i["field"].shape))
        g.load_particles(torch.from_numpy(i["xyz"]).to("cuda:0"), torch.from_numpy(i["attr"]).to("cuda:0"))
        _check(g, i)
    finally:
        g.close()
