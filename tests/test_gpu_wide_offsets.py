"""GPU: the kernels with 64-bit array offsets against those with 32-bit ones, in every storage, on a lattice
that needs neither (rows longer than a wave, periodic faces, inlet and outflow planes).

Each call gets the same inputs in both forms, and both run the same expressions, which the compiler may fuse
in another order. Tolerance per call, relative to the largest entry: 1e-10 in 64 bits, as in the parity
tests, 1e-4 in 32 bits (about 1e3 roundings of 6e-8); an offset that goes astray is off by the values
themselves. Stored 2-byte deviations may differ by their last bit (relative 2^-10 or 2^-7 of the largest).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4, "fp16": 1e-4 + 2.0 ** -10, "bf16": 1e-4 + 2.0 ** -7}


@pytest.fixture(scope="module")
def core():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_15781_amd import core as c

    c.lib()
    return c


def _close(name, a, b, tol):
    a, b = a.double().cpu().numpy(), b.double().cpu().numpy()
    top = np.abs(b).max()
    err = np.abs(a - b).max()
    print(name, "%.1e of %.1e" % (err, top), flush=True)
    assert np.isfinite(b).all() and err <= tol * top, (name, err, top)


@pytest.mark.parametrize("species", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
def test_wide_offsets_equal_narrow_ones(core, precision, species):
    import torch

    shape = (67, 14, 11)
    rng = np.random.default_rng(21)
    solid = (rng.uniform(size=shape[::-1]) < 0.3).astype(np.uint8)
    red = (rng.uniform(size=solid.shape) > 0.4).astype(np.float64)
    theta = rng.uniform(0.6, 2.4, solid.shape)

    def make(wide):
        sim = core.Lbm(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, precision=precision, tau=0.8,
                       sigma=0.02, beta=0.7, xi=0.02, accel=[(1e-5, 0, 0), (1e-5, 0, 0)], species=species, x_open=species,
                       tau_species=0.9)
        if wide:
            sim.use_wide_offsets()
        return sim

    narrow, wide = make(False), make(True)
    tol = TOL[precision]
    narrow.step(4)
    start = narrow.get_state()
    for sim in (narrow, wide):
        sim.set_state(start, 4)
    sums = [sim.step(1) for sim in (narrow, wide)]
    assert np.abs(sums[0] - sums[1]).max() <= 1e-6 * np.abs(sums[0]).max()
    (sa, sb) = (sim.state_sums(start) for sim in (narrow, wide))
    assert all(abs(sa[k] - sb[k]) <= 1e-12 * max(1.0, abs(sa[k])) for k in sa)
    for name, a, b in zip(("f^r", "f^p", "g"), wide.populations(), narrow.populations()):
        if name != "g" or species:
            _close(name, a, b, tol)
    for sim in (narrow, wide):
        sim.set_state(start, 4)
    ma, mb = wide.moments(), narrow.moments()
    for key in ("rho_r", "rho_p", "rho_n", "u") + (("c",) if species else ()):
        _close(key, ma[key], mb[key], tol)
    # kept fields and two adjoint steps, each from the 32-bit form's inputs
    fields = {}
    for name, sim in (("narrow", narrow), ("wide", wide)):
        fields[name] = sim.new_fields()
        sim.step_from(start, sim.new_state(), fields[name])
    lam = narrow.new_adjoint()
    narrow.adjoint_seed(start, lam)
    lam_wide = wide.new_adjoint()
    wide.adjoint_seed(start, lam_wide)
    _close("seed", lam_wide, lam, tol)
    tol = 1e-10 if precision == "fp64" else 1e-4  # adjoint states keep the arithmetic type
    F = narrow.nfluid
    for step in range(2):
        out, theta_grads, xi_grads = {}, {}, {}
        for name, sim in (("narrow", narrow), ("wide", wide)):
            for kept in (False, True):
                k = (name, kept)
                out[k] = sim.new_adjoint()
                theta_grads[k], xi_grads[k] = sim.new_gradients()
                sim.adjoint_step(start, lam, out[k], sim.new_scratch(), theta_grads[k], xi_grads[k],
                                 fields=fields[name] if kept else None)
        torch.cuda.synchronize()
        planes = slice(0, 30 if species else 23)
        for kept in (False, True):
            a, b = ("wide", kept), ("narrow", kept)
            _close("adjoint %d %d" % (step, kept), out[a][planes, :F], out[b][planes, :F], tol)
            _close("dL/dtheta", theta_grads[a], theta_grads[b], tol)
            _close("dL/dxi", xi_grads[a], xi_grads[b], tol)
        lam = out[("narrow", True)].clone()
