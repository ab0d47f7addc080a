"""GPU: the static geometry on axes of one to six nodes (shorter and longer than the stencils), against
periodic shifts of the mask. Link bits and flags are whole numbers; the wall normal is an exact
integer sum normalised once in FP64, which leaves a few roundings (1e-14)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def core():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_15781_amd import core as c

    c.lib()
    return c


def _at(a, c):
    """a at x + c for every x (arrays are indexed z, y, x)."""
    return np.roll(a, shift=(-c[2], -c[1], -c[0]), axis=(0, 1, 2))


@pytest.mark.parametrize("shape", [(1, 6, 5), (2, 1, 6), (3, 2, 1), (4, 3, 2), (5, 4, 3), (6, 5, 4), (67, 3, 2), (2, 66, 3), (1, 1, 1)])
@pytest.mark.parametrize("x_open", [False, True])
def test_geometry_on_short_axes(core, shape, x_open):
    import oracle

    if x_open and shape[0] < 2:
        pytest.skip("an open x axis has at least two nodes")
    rng = np.random.default_rng(sum(shape))
    solid = (rng.uniform(size=shape[::-1]) < 0.5).astype(np.uint8)
    solid[0, 0, 0] = 0
    theta = rng.uniform(0.6, 2.4, solid.shape)
    one = np.ones(solid.shape)
    sim = core.Lbm(shape, solid=solid, theta=theta, rho_r0=one, rho_p0=0 * one, xi=0.01, precision="fp64", tau=0.8,
                   tau_species=0.9, sigma=0.02, beta=0.7, accel=[(0, 0, 0)] * 2, species=True, x_open=x_open)
    info, wet = sim.geometry()
    info = info.cpu().numpy().astype(np.int64).reshape(solid.shape) & 0xFFFFFFFF
    wet = wet.cpu().numpy().reshape((4,) + solid.shape)
    c, _, _ = oracle.lattice()
    fluid = solid == 0
    want = np.zeros_like(info)
    for i in range(18):
        want |= np.where(fluid, _at(solid, -c[i]) != 0, _at(solid, c[i]) == 0).astype(np.int64) << i
    linked = want != 0
    nn = sum((_at(solid, c[i]) != 0).astype(np.int64) for i in range(6))
    want |= np.where(fluid, (1 << 18) | (linked.astype(np.int64) << 19) | (nn << 20), linked.astype(np.int64) << 23)
    if x_open:
        want[:, :, 0] |= np.where(fluid[:, :, 0], 1 << 24, 0)
        want[:, :, -1] |= np.where(fluid[:, :, -1], 1 << 25, 0)
    assert int((info != want).sum()) == 0
    e, w = oracle.e8()
    units = np.rint(5040 * w).astype(np.int64)
    s = np.stack([sum(int(k) * int(d[a]) * _at(solid, d).astype(np.int64) for d, k in zip(e, units)) for a in range(3)])
    s = s * (fluid & linked)
    length = np.sqrt((s * s).sum(0).astype(np.float64))
    normal = s / np.where(length > 0, length, 1)
    assert float(np.abs(wet[:3] - normal).max()) < 1e-14
    assert float(np.abs(wet[3] - np.where(fluid, np.cos(theta), 0)).max()) < 1e-15
