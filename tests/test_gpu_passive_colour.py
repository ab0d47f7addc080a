"""GPU: the one-kernel step taken when neither the force nor the recolouring uses a normal
(sigma = beta = 0), against the oracle and against the general passes of the kept-fields step.

Tolerance: FP64 arithmetic on both sides, as in the parity tests; the two GPU paths share every
expression, so they agree to the last bit.
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


def _problem(shape, two_colours, species, porosity, seed):
    rng = np.random.default_rng(seed)
    solid = (rng.uniform(size=shape[::-1]) > porosity).astype(np.uint8)
    red = (rng.uniform(size=solid.shape) > 0.4).astype(np.float64) if two_colours else np.ones(solid.shape)
    kw = dict(tau=0.8, sigma=0.0, beta=0.0, accel=[(1e-5, 0, 0), (0, 2e-5, 0)], species=species, x_open=species)
    return solid, red, kw


@pytest.mark.parametrize("shape,porosity", [((2, 5, 3), 1.0), ((17, 9, 7), 0.5), ((33, 16, 16), 0.7), ((64, 17, 9), 0.9)])
@pytest.mark.parametrize("two_colours,species,xi", [(False, False, 0.0), (True, False, 0.02), (True, True, 0.02)])
def test_passive_colour_matches_oracle(core, shape, porosity, two_colours, species, xi):
    import oracle

    solid, red, kw = _problem(shape, two_colours, species, porosity, 11)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=xi, precision="fp64", tau_species=0.9, **kw)
    ref = oracle.Oracle(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=xi, tau_c=0.9, **kw)
    sums, rsums = sim.step(15), ref.step(15)
    assert np.abs(sums[:, :4] - rsums[:, :4]).max() <= FP64_TOL * np.abs(rsums[:, :4]).max()
    assert not sums[:, 4].any()
    m, r = sim.moments(), ref.moments()
    for key in ("rho_r", "rho_p", "rho_n", "u") + (("c",) if species else ()):
        err, top = float(np.abs(m[key].cpu().numpy() - r[key]).max()), float(np.abs(r[key]).max())
        assert err <= FP64_TOL * top, (key, err, top)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
def test_passive_colour_step_equals_general_passes(core, precision):
    import torch

    shape = (33, 12, 10)
    solid, red, kw = _problem(shape, True, True, 0.7, 13)
    sim = core.Lbm(shape, solid=solid, rho_r0=red, rho_p0=1 - red, xi=0.01, precision=precision, tau_species=0.9, **kw)
    sim.step(5)
    start = sim.get_state()
    out, plain, fields = sim.new_state(), sim.new_state(), sim.new_fields()
    sim.step_from(start, out, fields)
    sim.step_from(start, plain)
    sim.step(1)
    got = sim.get_state()
    for a in (out, plain):
        if precision in ("fp64", "fp32"):
            assert all(torch.equal(x, y) for x, y in zip(sim.state_parts(a), sim.state_parts(got)))
    sim.set_state(out, 6)
    kept = sim.populations()
    sim.set_state(got, 6)
    assert all(torch.equal(x, y) for x, y in zip(kept, sim.populations()))
