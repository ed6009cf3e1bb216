"""Persistent rounds on dense features: the blocks that take part follow the
coupled steps, so a pull of millions of them is not left to a few blocks, and the
masks are those of launched rounds."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


def _dense(X, Y, Z, T, P, frac):
    """A smooth field moving along x, particles drifting in it with its values,
    and the threshold that admits `frac` of the field."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    c = torch.rand((1, 1, Z // 8, Y // 8, X // 8), device=DEV, generator=gen)
    a = torch.nn.functional.interpolate(c, size=(Z, Y, X), mode="trilinear")[0, 0]
    f = torch.stack([torch.roll(a, t, 2) for t in range(T)])
    size = torch.tensor([X, Y, Z], device=DEV, dtype=torch.float32)
    p0 = torch.rand((P, 3), device=DEV, generator=gen) * size
    v = (torch.rand((P, 3), device=DEV, generator=gen) - 0.5) * 0.5
    xyz = torch.stack([torch.minimum(torch.remainder(p0 + v * t, size), size - 0.01) for t in range(T)])
    i = xyz.long()
    t = torch.arange(T, device=DEV)[:, None]
    attr = f[t, i[..., 2], i[..., 1], i[..., 0]].contiguous()
    k = int(a.argmax())
    tau = float(torch.quantile(f[0].reshape(-1)[::7].contiguous(), 1.0 - frac))
    return f, xyz, attr, tau, np.array([[k % X, k // X % Y, k // (X * Y), 0]], np.int32)


def _grow(schedule, data, bt, reps):
    from paper_1903_12294_amd import Grower
    f, xyz, attr, tau, seeds = data
    T, P = attr.shape
    g = Grower(device=0, tile_t=bt, schedule=schedule)
    try:
        g.load_field(f)
        g.load_particles(xyz, attr)
        fm = torch.zeros((f.numel() + 31) // 32, dtype=torch.int32, device=DEV)
        pm = torch.zeros((T, P), dtype=torch.uint8, device=DEV)
        times = []
        for _ in range(reps):
            g.set_criteria(tau, np.inf, tau, np.inf)
            g.set_seeds(seeds)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            g.grow_read(fm, pm)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return fm, pm, float(np.median(times[2:]))
    finally:
        g.close()


# tile depth 8 at 128^3 x 32: 64 blocks by the tiles, 2,000 and more by the steps;
# 96 x 96 x 64 x 9 at depth 16: 24 by the tiles (one depth whose last tiles are ragged)
@pytest.mark.parametrize("dims,P,bt,frac", [((128, 128, 128, 32), 262144, 8, 0.3), ((96, 96, 64, 9), 60001, 16, 0.9)])
def test_dense_feature_uses_the_grid(dims, P, bt, frac):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    data = _dense(*dims, P, frac)
    print(f"[grid] {dims} launch", flush=True)
    fl, pl, tl = _grow("launch", data, bt, 9)
    print(f"[grid] {dims} persistent", flush=True)
    fp, pp, tp = _grow("persistent", data, bt, 9)
    assert torch.equal(fl, fp) and torch.equal(pl, pp)
    assert int(pl.sum()) > P  # dense indeed
    # both run the same phases; the barriers between them cost tens of
    # microseconds a round, too few blocks several times the whole
    print(f"[grid] launch {tl * 1e6:.0f} us, persistent {tp * 1e6:.0f} us", flush=True)
    assert tp < 2.5 * tl
