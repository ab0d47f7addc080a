"""GPU: the step's FP64 sums across workgroup, wave and chunk edges, and the read-out at solid nodes.

Sums are compared with the oracle's at the parity tests' tolerance (both sides add the same FP64
terms, in different orders), and between one call and many to the last bit (the same additions).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-10


@pytest.fixture(scope="module")
def core():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_15781_amd import core as c

    c.lib()
    return c


def _sim(core, shape, porosity=0.6, **kw):
    rng = np.random.default_rng(3)
    solid = (rng.uniform(size=shape[::-1]) > porosity).astype(np.uint8)
    red = (rng.uniform(size=solid.shape) > 0.4).astype(np.float64)
    args = dict(tau=0.8, sigma=0.02, beta=0.7, accel=[(1e-5, 0, 0)] * 2, species=True, x_open=shape[0] > 1)
    args.update(kw)
    return solid, red, args


# fluid nodes below, at and above one wave, one workgroup and the eight workgroups of a round
@pytest.mark.parametrize("shape", [(2, 1, 1), (7, 3, 3), (64, 1, 1), (5, 13, 1), (16, 16, 1), (257, 1, 1), (32, 8, 8), (2049, 1, 1)])
@pytest.mark.parametrize("sigma,beta", [(0.02, 0.7), (0.0, 0.0)])
def test_sums_match_oracle(core, shape, sigma, beta):
    import oracle

    solid, red, kw = _sim(core, shape, porosity=1.0, sigma=sigma, beta=beta)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, precision="fp64", tau_species=0.9, **kw)
    ref = oracle.Oracle(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, tau_c=0.9, **kw)
    got, want = sim.step(3), ref.step(3)
    assert np.abs(got[:, :4] - want[:, :4]).max() <= FP64_TOL * np.abs(want[:, :4]).max()
    assert not got[:, 4].any()


@pytest.mark.parametrize("sigma,beta", [(0.02, 0.7), (0.0, 0.0)])
def test_sums_do_not_depend_on_the_call(core, sigma, beta):
    import torch

    shape, n = (24, 10, 9), 1030  # past the 1024 rows kept on the device
    solid, red, kw = _sim(core, shape, sigma=sigma, beta=beta)
    sims = [core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=1e-3, precision="fp32", tau_species=0.9, **kw)
            for _ in range(3)]
    whole = sims[0].step(n)
    parts = np.concatenate([sims[1].step(k) for k in (1, 1, 2, 500, 26, 499, 1)])
    sims[2].advance(n)
    assert np.array_equal(whole, parts)
    first = [p.cpu() for p in sims[0].populations()]
    for other in sims[1:]:
        assert all(torch.equal(a, b.cpu()) for a, b in zip(first, other.populations()))


def test_nonfinite_nodes_are_counted(core):
    shape = (20, 8, 8)
    solid, red, kw = _sim(core, shape, porosity=1.0)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.0, precision="fp64", tau_species=0.9, **kw)
    state = sim.get_state()
    f, _, _ = sim.state_parts(state)
    f[18, [3, 700, 1200]] = float("nan")  # rest populations: pulled by their own nodes only
    sim.set_state(state, 0)
    sums = sim.step(1, check=False)
    assert sim.last_status == core.LBM_ERR_NONFINITE
    assert sums[0, 4] >= 3
    assert sim.state_sums(state)["nonfinite"] == 3


def test_moments_write_zero_at_solid_nodes(core):
    import torch

    shape = (37, 11, 5)
    solid, red, kw = _sim(core, shape)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, precision="fp32", tau_species=0.9, **kw)
    N = solid.size
    out = [torch.full((k * N,), float("nan"), device="cuda:0") for k in (1, 1, 1, 3, 1)]
    lib = core.lib()
    assert lib.lbm_moments(sim._h, *[t.data_ptr() for t in out]) == 0
    torch.cuda.synchronize()
    flat = torch.as_tensor(solid.reshape(-1), device="cuda:0").bool()
    for t in out:
        t = t.view(-1, N)
        assert torch.isfinite(t).all()
        assert (t[:, flat] == 0).all()
    # any of the outputs may be absent
    only = torch.full((3 * N,), float("nan"), device="cuda:0")
    assert lib.lbm_moments(sim._h, None, None, None, only.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(only, out[3])


# a cube of each way to share tiles among workgroups, and the node counts on both sides of the lines between
@pytest.mark.parametrize("shape,precision", [((32, 32, 32), "fp64"), ((32, 32, 33), "fp64"), ((64, 32, 32), "fp64"),
                                             ((41, 40, 40), "fp64"), ((32, 32, 32), "fp32"), ((32, 32, 33), "fp32"),
                                             ((128, 48, 32), "fp32"), ((128, 48, 33), "fp32")])
def test_sums_and_fields_at_the_workgroup_sizes(core, shape, precision):
    """Three steps against the oracle. FP64 as above. FP32 storage: the populations of a node are
    rounded once a step (6e-8 relative) and its arithmetic adds a few dozen roundings, none of which
    grows in three steps, so 2e-5 of the largest value leaves two orders over their sum."""
    import oracle

    tol = FP64_TOL if precision == "fp64" else 2e-5
    solid, red, kw = _sim(core, shape, porosity=1.0)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, precision=precision, tau_species=0.9, **kw)
    ref = oracle.Oracle(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, tau_c=0.9, **kw)
    got, want = sim.step(3), ref.step(3)
    assert np.abs(got[:, :4] - want[:, :4]).max() <= tol * np.abs(want[:, :4]).max()
    assert not got[:, 4].any()
    for k, (a, b) in enumerate(zip(sim.populations(), ref.get_state())):
        err, bound = float(np.abs(a.cpu().numpy() - b).max()), tol * float(np.abs(b).max())
        assert err <= bound, (k, err, bound)
