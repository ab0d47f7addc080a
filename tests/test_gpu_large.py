"""GPU: what only large lattices use (nontemporal stores, the launch order of many tiles) against a small
lattice, which does without. The large lattice repeats the small one, so each node goes through the
same arithmetic and the fields are equal to the last bit; the FP64 sums add the same terms in another
order (1e-12 relative)."""
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


# fluid nodes on both sides of the lines: two states of 248 and 370 MB with species, of 320 MB without, 4.2 million nodes
@pytest.mark.parametrize("precision,reps,species,sigma", [
    ("fp64", (3, 3, 2), True, 0.01), ("fp64", (3, 3, 3), True, 0.01), ("fp64", (3, 4, 3), False, 0.0),
    ("fp32", (4, 3, 3), True, 0.01), ("fp32", (6, 3, 3), True, 0.01), ("fp32", (5, 5, 5), False, 0.01),
    ("fp32", (6, 5, 5), True, 0.0), ("fp16", (5, 5, 5), True, 0.01), ("fp16", (6, 5, 5), False, 0.01),
    ("bf16", (7, 3, 3), True, 0.01), ("bf16", (6, 5, 5), True, 0.01)])
def test_large_lattice_equals_its_tile(core, precision, reps, species, sigma):
    import torch

    tile = (36, 33, 31)
    rng = np.random.default_rng(11)
    solid = (rng.uniform(size=tile[::-1]) < 0.08).astype(np.uint8)
    red = (rng.uniform(size=solid.shape) > 0.5).astype(np.float64)
    kw = dict(tau=0.8, sigma=sigma, beta=70 * sigma, xi=1e-3, accel=[(1e-5, 0, 0), (1e-5, 0, 0)], precision=precision,
              species=species, tau_species=0.9, theta_uniform=1.0)

    def run(rep):
        s, r = (np.tile(a, rep[::-1]) for a in (solid, red))
        sim = core.Lbm(tuple(a * k for a, k in zip(tile, rep)), solid=s, rho_r0=r, rho_p0=1 - r, **kw)
        sums = sim.step(3)
        m = sim.moments()
        return sums, m

    small_sums, small = run((1, 1, 1))
    sums, big = run(reps)
    want = small_sums[:, :4] * np.prod(reps)
    assert np.abs(sums[:, :4] - want).max() <= 1e-12 * np.abs(want).max() and not sums[:, 4].any()
    for key, one in small.items():
        got = big.pop(key)
        for z in range(reps[2]):
            part = got[..., z * tile[2]:(z + 1) * tile[2], :, :]
            assert torch.equal(part, one.repeat(*([1] * (one.dim() - 2)), reps[1], reps[0])), (key, z)
        del got
    torch.cuda.empty_cache()
