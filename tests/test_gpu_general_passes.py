"""GPU: the branches that leave work out, against the passes that do it and against the oracle.

The one-kernel step (sigma = beta = 0) is compared with the four passes of a second context whose sigma is
1e-300: not zero on the host, so that the passes run, and without effect on any sum (zero in 32-bit
arithmetic). Both evaluate the same expressions on the same inputs, which the compiler may fuse in another
order. Tolerances for one step, relative to the largest entry: 1e-12 in 64 bits and 1e-5 in 32 bits (a few
dozen roundings of 2e-16 and 6e-8); 2-byte populations may also differ by the last bit of a deviation,
2^-11 or 2^-8 of the largest of them, itself below the largest population.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5, "fp16": 1e-5 + 2.0 ** -11, "bf16": 1e-5 + 2.0 ** -8}


@pytest.fixture(scope="module")
def core():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_15781_amd import core as c

    c.lib()
    return c


def _mixture(shape, seed):
    rng = np.random.default_rng(seed)
    solid = (rng.uniform(size=shape[::-1]) < 0.3).astype(np.uint8)
    return solid, rng.uniform(0.05, 0.95, solid.shape), rng.uniform(0.6, 2.4, solid.shape)


def _passive(core, shape, sigma, precision, species, seed=13):
    solid, red, theta = _mixture(shape, seed)
    kw = dict(tau=0.8, sigma=sigma, beta=0.0, accel=[(1e-5, 0, 0), (0, 2e-5, 0)], species=species, x_open=species)
    sim = core.Lbm(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, xi=0.02, precision=precision,
                   tau_species=0.9, **kw)
    return sim, solid, red, theta, kw


@pytest.mark.parametrize("species", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
def test_one_kernel_step_equals_the_four_passes(core, precision, species):
    import torch

    shape = (67, 12, 10)
    one, solid, *_ = _passive(core, shape, 0.0, precision, species)
    four, *_ = _passive(core, shape, 1e-300, precision, species)
    one.step(6, reductions=False)
    start = one.get_state()
    four.set_state(start, 6)
    tol = TOL[precision]
    got, want = one.step(1), four.step(1)
    scale = np.abs(want[:, :4]).max()
    assert np.abs(got[:, :4] - want[:, :4]).max() <= min(tol, 1e-5) * scale
    parts = list(zip(("f^r", "f^p", "g"), one.populations(), four.populations()))
    for sim in (one, four):
        sim.set_state(start, 6)
    a, b = one.moments(), four.moments()
    parts += [(k, a[k], b[k]) for k in ("rho_r", "rho_p", "rho_n", "u") + (("c",) if species else ())]
    for name, x, y in parts[:2] + parts[2 if species else 3:]:
        err, top = float((x - y).abs().max()), float(y.abs().max())
        print(precision, species, name, "%.1e of %.1e" % (err, top), flush=True)
        assert err <= tol * top, (name, err, top)
    # fields kept beside the one-kernel step are those of the passes, which both contexts run alike
    kept = []
    for sim in (one, four):
        f = sim.new_fields().zero_()
        sim.step_from(start, sim.new_state(), f)
        torch.cuda.synchronize()
        kept.append(f)
    real = one.real
    n = one.N * (8 if precision == "fp64" else 4)
    q = [f[:n].view(real) for f in kept]
    assert torch.equal(q[0], q[1])
    fluid = torch.as_tensor(solid.reshape(-1) == 0, device="cuda:0")
    rho_n = q[0] + torch.where(torch.signbit(q[0]), 1.0, -1.0).to(real)  # kept as the offset from the nearer pure state
    err = float((rho_n - b["rho_n"].reshape(-1))[fluid].abs().max())
    assert err <= tol, err


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 2e-5)])
def test_one_kernel_step_and_its_fields_match_the_oracle(core, precision, tol):
    """Three steps; tolerances as in the tests of the sums (64 and 32 bits)."""
    import oracle
    import torch

    shape = (33, 12, 10)
    sim, solid, red, theta, kw = _passive(core, shape, 0.0, precision, True, seed=17)
    ref = oracle.Oracle(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, xi=0.02, tau_c=0.9, **kw)
    got, want = sim.step(3), ref.step(3)
    assert np.abs(got[:, :4] - want[:, :4]).max() <= tol * np.abs(want[:, :4]).max()
    for k, (a, b) in enumerate(zip(sim.populations(), ref.get_state())):
        assert float(np.abs(a.cpu().numpy() - b).max()) <= tol * float(np.abs(b).max()), k
    fields = sim.new_fields()
    sim.step_from(sim.get_state(), sim.new_state(), fields)
    torch.cuda.synchronize()
    q = fields[:sim.N * (8 if precision == "fp64" else 4)].view(sim.real).double().cpu().numpy()
    rho_n = q + np.where(np.signbit(q), 1.0, -1.0)
    fluid = solid.reshape(-1) == 0
    assert np.abs(rho_n - ref.moments()["rho_n"].reshape(-1))[fluid].max() <= tol


@pytest.mark.parametrize("sigma,beta", [(0.0, 0.0), (0.0, 0.7), (0.02, 0.0)])
def test_gradient_without_force_or_recolouring(core, oracle_mod, sigma, beta):
    """Against the oracle's duals, and bit for bit between the ways to keep the levels and their fields."""
    import torch

    from paper_2608_15781_amd import autograd as ag

    shape, xi, T = (11, 9, 8), 0.05, 18
    solid, red, theta = _mixture(shape, 23)
    red = red * (1 - solid)
    kw = dict(tau=0.7, sigma=sigma, beta=beta, accel=[(2e-5, 0, 0), (2e-5, 0, 0)], species=True, x_open=True)
    rng = np.random.default_rng(24)
    d = rng.normal(size=solid.shape) * (1 - solid)
    rp0 = (1 - solid) - red
    L, dL = oracle_mod.grad(shape, solid, theta, xi, T, dtheta=[d.ravel(), np.zeros(solid.size)], dxi=[0.0, 1.0],
                            rho_r0=red, rho_p0=rp0, tau_c=0.8, **kw)

    def make():
        return core.Lbm(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=rp0, xi=xi, precision="fp64", tau_species=0.8, **kw)

    sim = make()
    Lg, cps, final = ag.forward_states(sim, T, 7)
    gth, gxi, _ = ag.adjoint_gradients(sim, T, 7, cps, final)
    assert abs(Lg - L) <= 1e-10 * abs(L)
    ad = [float(gth.cpu().numpy() @ d.ravel()), float(gxi)]
    print("adjoint", ad, "duals", list(dL), flush=True)
    for a, b in zip(ad, dL):
        assert abs(a - b) <= 1e-8 * abs(b) + 1e-14, (a, b)
    if sigma == 0 and beta == 0:
        assert not gth.any()
    again, gxi2, _ = ag.adjoint_gradients(sim, T, 7, cps, final, keep_fields=False)
    assert torch.equal(again, gth) and float(gxi2) == float(gxi)
    sim = make()
    L3, levels, last = ag.forward_keep_all(sim, T)
    all_th, all_xi, _ = ag.adjoint_gradients_keep_all(sim, levels, last)
    assert torch.equal(all_th, gth) and float(all_xi) == float(gxi) and abs(L3 - Lg) <= 1e-11 * abs(Lg)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("interface", [False, True])
def test_nonfinite_nodes_spread_as_in_the_oracle(core, precision, value, interface):
    """One non-finite rest population: the same nodes are non-finite after one step and after two, whether or not
    its wave has a node with |G| > eps (a uniform mixture has none: |G| is not a number round the node and
    the curvature gathers are skipped)."""
    import oracle

    shape = (40, 9, 8)
    solid = np.zeros(shape[::-1], np.uint8)
    solid[:, 0, :] = 1
    red = np.full(solid.shape, 0.5)
    if interface:
        red[:, :, 18:] = 0.3
    kw = dict(tau=0.8, sigma=0.02, beta=0.7, accel=[(0, 0, 0)] * 2, species=False)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, precision=precision, **kw)
    ref = oracle.Oracle(shape, solid=solid, rho_r0=red, rho_p0=1 - red, **kw)
    node = 20 + 40 * (4 + 9 * 4)
    rank = int((solid.reshape(-1)[:node] == 0).sum())
    state = sim.get_state()
    sim.state_parts(state)[0][18, rank] = value
    sim.set_state(state, 0)
    fr, fp, _ = ref.get_state()
    fr[18, node] = fp[18, node] = value
    ref.set_state(fr, fp)
    for step in range(2):
        sums = sim.step(1, check=False)
        ref.step(1)
        got = [~np.isfinite(t.cpu().numpy()).all(axis=0) for t in sim.populations()[:2]]
        want = [~np.isfinite(t).all(axis=0) for t in ref.get_state()[:2]]
        print(precision, value, interface, step, int(got[0].sum()), int(want[0].sum()), flush=True)
        assert want[0].sum() >= 19
        assert (got[0] == want[0]).all() and (got[1] == want[1]).all()
        assert sums[0, 4] == (got[0] | got[1]).sum()
