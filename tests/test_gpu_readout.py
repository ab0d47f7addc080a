"""GPU: read-outs over node counts round the 32-node words of the id map and the workgroups, and over solid
fractions on both sides of the line between the two ways to clear a field."""
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


def _sim(core, shape, nsolid, precision="fp64", seed=7, **kw):
    rng = np.random.default_rng(seed)
    solid = np.zeros(int(np.prod(shape)), np.uint8)
    solid[rng.permutation(solid.size)[:nsolid]] = 1
    theta = rng.uniform(0.6, 2.4, solid.size)
    red = rng.uniform(0.1, 0.9, solid.size)
    sim = core.Lbm(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, precision=precision, tau=0.8,
                   species=True, c0=rng.uniform(0.2, 1.0, solid.size), **dict(dict(sigma=0.02, beta=0.7), **kw))
    return solid.astype(bool), theta, sim


# none, one, a fifth, one more than a fifth, all but one and all of 300 nodes
@pytest.mark.parametrize("nsolid", [0, 1, 60, 61, 299, 300])
@pytest.mark.parametrize("sigma,beta", [(0.02, 0.7), (0.0, 0.0)])
def test_fields_are_zero_at_solids_and_written_at_fluid_nodes(core, nsolid, sigma, beta):
    import torch

    shape, N = (25, 6, 2), 300
    solid, _, sim = _sim(core, shape, nsolid, sigma=sigma, beta=beta)
    want = sim.moments()
    fluid = torch.as_tensor(~solid, device="cuda:0")
    # outputs that start at any element, filled with what must not survive
    store = [torch.full((k * N + 3,), float("nan"), dtype=torch.float64, device="cuda:0") for k in (1, 1, 1, 3, 1)]
    out = [t[1 + (j % 2):][:t.numel() - 3] for j, t in enumerate(store)]
    assert core.lib().lbm_moments(sim._h, *[t.data_ptr() for t in out]) == 0
    torch.cuda.synchronize()
    for t, key in zip(out, ("rho_r", "rho_p", "rho_n", "u", "c")):
        t, w = t.view(-1, N), want[key].reshape(-1, N)
        assert torch.isfinite(t).all() and torch.equal(t, w), key
        assert (t[:, ~fluid] == 0).all(), key
        if key in ("rho_r", "rho_p", "c"):
            assert (t[:, fluid] > 0).all(), key
    for j, t in enumerate(store):  # nothing outside the outputs
        assert torch.isnan(t[:1 + (j % 2)]).all() and torch.isnan(t[1 + (j % 2) + t.numel() - 3:]).all()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx", [1, 31, 32, 33, 255, 256, 257, 511, 512, 513, 1025])
def test_populations_and_geometry_follow_the_state(core, nx, precision):
    """The colours add up to the stored f^m (one rounding each of a f + k and b f - k: 4 units of the
    last place of the largest value), the species are the stored ones, and cos(theta) is the input's."""
    import torch

    eps = 2.2e-16 if precision == "fp64" else 1.2e-7
    for nsolid in {0, nx // 3, nx - 1}:
        solid, theta, sim = _sim(core, (nx, 1, 1), nsolid, precision=precision)
        fluid = torch.as_tensor(np.flatnonzero(~solid), device="cuda:0")
        f, _, g = sim.state_parts(sim.get_state())
        fr, fp, go = sim.populations()
        assert float((fr[:, fluid] + fp[:, fluid] - f).abs().max()) <= 4 * eps * float(f.abs().max())
        assert torch.equal(go[:, fluid], g)
        info, wet = sim.geometry()
        assert np.abs(wet[3, fluid].double().cpu().numpy() - np.cos(theta[~solid])).max() <= 2 * eps
        bad = torch.as_tensor(np.flatnonzero(solid), device="cuda:0")
        for t in (fr, fp, go, wet):
            assert (t[:, bad] == 0).all()
        assert ((info.cpu().numpy() >> 18 & 1).astype(bool) == ~solid).all()
