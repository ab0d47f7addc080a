"""GPU: the pull-source map, the shared row gathers and the two offset widths at their edges.

The oracle comparison runs masks made of short runs of fluid nodes (single nodes with no fluid
neighbour along the row, runs that end at a wave's last lane, rows whose centre is solid) at row
lengths on both sides of the map's 32-node words and the 64-wide wave. Tolerance: FP64 arithmetic on
both sides, as in the parity tests. The wide-offset comparison tiles a small lattice: every tile of
the large one goes through the same arithmetic per node, so the fields are equal to the last bit.
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


@pytest.mark.parametrize("species", [False, True])
@pytest.mark.parametrize("nx", [1, 2, 3, 31, 32, 33, 64, 65, 129])
def test_short_runs_match_oracle(core, nx, species):
    import oracle

    shape = (nx, 9, 7)
    rng = np.random.default_rng(100 + nx)
    solid = (rng.uniform(size=shape[::-1]) < 0.55).astype(np.uint8)
    solid[3, 4, :] = 0  # a row without any solid node
    theta = rng.uniform(0.6, 2.4, solid.shape)
    red = (rng.uniform(size=solid.shape) > 0.4).astype(np.float64)
    kw = dict(tau=0.8, sigma=0.02, beta=0.7, accel=[(1e-5, 0, 0), (1e-5, 0, 0)], species=species,
              x_open=species and nx > 1)
    sim = core.Lbm(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, xi=0.01, precision="fp64",
                   tau_species=0.9, **kw)
    ref = oracle.Oracle(shape, solid=solid, theta=theta, rho_r0=red, rho_p0=1 - red, xi=0.01, tau_c=0.9, **kw)
    red_sums, ref_sums = sim.step(12), ref.step(12)
    assert np.abs(red_sums[:, :4] - ref_sums[:, :4]).max() <= FP64_TOL * np.abs(ref_sums[:, :4]).max()
    m, r = sim.moments(), ref.moments()
    for key in ("rho_r", "rho_p", "rho_n", "u") + (("c",) if species else ()):
        err = np.abs(m[key].cpu().numpy() - r[key]).max() / np.abs(r[key]).max()
        print(nx, species, key, "%.1e" % err, flush=True)
        assert err < FP64_TOL, (key, err)
    for k, (got, want) in enumerate(zip(sim.populations(), ref.get_state())):
        if k == 2 and not species:
            continue
        err = float(np.abs(got.cpu().numpy() - want).max())
        bound = FP64_TOL * float(np.abs(want).max())
        assert err <= bound, (k, err, bound)


@pytest.mark.parametrize("species", [False, True])
def test_wide_offsets_equal_narrow_ones(core, species):
    """92 million FP64 nodes pass the 32-bit offsets; the lattice repeats a 32^3 one 15 x 14 x 14 times."""
    import torch

    tile, reps = 32, (15, 14, 14)
    rng = np.random.default_rng(5)
    solid = np.zeros((tile,) * 3, np.uint8)
    solid[rng.integers(0, tile, 40), rng.integers(0, tile, 40), rng.integers(0, tile, 40)] = 1
    red = (rng.uniform(size=solid.shape) > 0.5).astype(np.float64)
    kw = dict(tau=0.8, sigma=0.01, beta=0.7, xi=1e-3, accel=[(1e-5, 0, 0), (1e-5, 0, 0)], precision="fp64",
              species=species, tau_species=0.9, theta_uniform=1.0)

    def run(rep):
        s, r = (np.tile(a, rep[::-1]) for a in (solid, red))
        sim = core.Lbm(tuple(tile * k for k in rep), solid=s, rho_r0=r, rho_p0=1 - r, **kw)
        sim.step(3, reductions=False)
        return sim.moments()

    small = run((1, 1, 1))
    big = run(reps)
    for key, want in small.items():
        got = big.pop(key)
        for z in range(reps[2]):
            part = got[..., z * tile:(z + 1) * tile, :, :]
            assert torch.equal(part, want.repeat(*([1] * (want.dim() - 2)), reps[1], reps[0])), (key, z)
        del got
    torch.cuda.empty_cache()
