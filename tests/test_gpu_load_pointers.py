"""Device pointers given to a load: one that a copy accepts loads (device memory,
aligned or not to 16 bytes, and pinned host memory), one whose allocation is too
short is refused on the host, and the context is usable afterwards."""
import ctypes

import numpy as np
import pytest

from oracle import oracle_grow
from paper_1903_12294_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _load(g, ptr, dims, T):
    X, Y, Z = dims
    return g.lib.mf4d_load_field(g.ctx, ctypes.c_void_p(ptr), X, Y, Z, T, 1)  # MF4D_DEVICE


def _check(g, inst):
    X, Y, Z = inst["dims"]
    g.dims, g.T, g.Tp, g.P = (X, Y, Z), inst["T"], inst["T"], 0
    g.set_criteria(*inst["crit"])
    g.set_seeds(inst["seeds"])
    g.grow()
    none = np.zeros((inst["T"], 0, 3), np.float32), np.zeros((inst["T"], 0), np.float32)
    assert np.array_equal(g.read_field_mask(), oracle_grow(inst["field"], *none, inst["crit"], inst["seeds"])[0])


def test_field_pointer_is_checked_before_a_kernel_reads_it():
    from paper_1903_12294_amd import Grower, _lib
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    inst = synth.make_instance(36, 20, 12, 8, 8, n_blobs=4, seed=5, n_seeds=4, tau_f=0.25, tau_p=0.25)
    f = torch.from_numpy(inst["field"])
    g = Grower(device=0)
    lib = _lib.load_library()
    held = lib.mf4d_device_bytes()
    short = ctypes.c_void_p()  # an allocation of its own (torch's lie in larger ones)
    assert lib.hipMalloc(ctypes.byref(short), ctypes.c_size_t(1 << 20)) == 0
    try:
        # 1 MiB read as a field of 4 MiB
        print("[pointers] too short", flush=True)
        assert _load(g, short.value, (128, 128, 16), 4) == _lib.MF4D_ERR_HIP
        assert "allocation ends" in lib.mf4d_last_error().decode()
        assert lib.mf4d_device_bytes() == held
        with pytest.raises(_lib.MF4DError) as err:
            g.grow()
        assert err.value.code == _lib.MF4D_ERR_STATE
        own = torch.zeros(f.numel() + 8, device="cuda:0")
        for off in (0, 1, 4):  # floats
            print(f"[pointers] device + {off}", flush=True)
            own[off:off + f.numel()].copy_(f.reshape(-1))
            assert _load(g, own.data_ptr() + 4 * off, inst["dims"], inst["T"]) == 0
            _check(g, inst)
        print("[pointers] the same sizes, too short", flush=True)
        assert _load(g, short.value + (1 << 20) - 256, inst["dims"], inst["T"]) == _lib.MF4D_ERR_HIP
        pinned = torch.empty(f.numel(), pin_memory=True)
        pinned.copy_(f.reshape(-1))
        print("[pointers] pinned", flush=True)
        assert _load(g, pinned.data_ptr(), inst["dims"], inst["T"]) == 0
        _check(g, inst)
    finally:
        g.close()
        assert lib.hipFree(short) == 0
