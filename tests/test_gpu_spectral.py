"""GPU parity of the spectral density kernel (variant code 136, the default of
the density kind) against the FP64 oracle: both ends of every padded band-window
size, every padded orbital count and one below it, frequency counts around the
group of 16, several k-points per work item, equal and nearly equal band
energies, projectors without orthonormal rows, each output alone, and lattices
whose padded sizes run different kernels.  1e-10 relative, normwise per k and
per frequency, as for the other variants."""
import numpy as np
import pytest

import oracle
from paper_1111_2157_amd import synth
from gpu_util import RTOL, assert_gloc_parity, assert_nk_parity, gpu_density, relerr

pytestmark = pytest.mark.gpu

SPEC = 136


@pytest.fixture(scope="module")
def ctx():
    from paper_1111_2157_amd.dyson import Context

    c = Context(0)
    for nbp in (16, 32, 48, 64):
        assert c.get_variant(0, nbp) == SPEC
    yield c
    c.close()


def check(c, wl, mu, tail=2, lat=None):
    lat = lat or wl.lattice
    mats, gl, sc = gpu_density(c, wl, mu, tail, lat=lat)
    assert_nk_parity(mats, lat, wl.sigma, mu, tail)
    assert_gloc_parity(gl, lat, wl.sigma, mu)
    n = sum(lat.wk[k] * np.trace(m).real for k, m in enumerate(mats))
    h = sum(lat.wk[k] * np.sum(lat.eps_k(k) * np.diag(m).real) for k, m in enumerate(mats))
    q = sum(lat.wk[k] * np.trace(lat.proj_k(k) @ m @ lat.proj_k(k).conj().T).real for k, m in enumerate(mats))
    assert np.abs(sc - [n, q, h]).max() <= RTOL * max(1.0, np.abs(sc).max())


@pytest.mark.parametrize("nb", [1, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("nc", [1, 4, 5, 6, 7, 9, 11, 14, 15, 16])
def test_band_and_orbital_edges(ctx, nb, nc):
    if nc > nb:
        pytest.skip("a window holds at least nc bands")
    print("spectral nb", nb, "nc", nc, flush=True)
    check(ctx, synth.f_shell(nk=3, nb=nb, nc=nc, nw=21, n_narrow=min(nb, nc)), 0.2)


@pytest.mark.parametrize("nw", [1, 3, 15, 16, 17, 33, 64])
@pytest.mark.parametrize("nc", [3, 10])
def test_frequency_groups(ctx, nw, nc):
    print("spectral nw", nw, nc, flush=True)
    check(ctx, synth.d_shell(nk=5, nb=30, nc=10, nw=nw) if nc == 10 else synth.plain(nk=5, nb=19, nc=nc, nw=nw), -0.3)


@pytest.mark.parametrize("tail", [0, 2])
def test_many_k_points_per_item(ctx, tail):
    """2500 k-points: the default tile walks several of them per work item, so the
    G_loc partial is added to after its first k-point."""
    wl = synth.plain(nk=2500, nb=9, nc=4, nw=18)
    mats, gl, sc = gpu_density(ctx, wl, 0.4, tail)
    ks = [0, 1, 7, 63, 64, 1249, 2498, 2499]
    assert_nk_parity(mats, wl.lattice, wl.sigma, 0.4, tail, klist=ks)
    assert_gloc_parity(gl, wl.lattice, wl.sigma, 0.4)


@pytest.mark.parametrize("nb,nc", [(24, 5), (40, 14), (64, 10)])
def test_equal_and_close_energies(ctx, nb, nc):
    """Pairs and a triple of equal energies, steps of 1e-13 to 1e-2 eV, a window
    with a single energy, energies in descending order."""
    wl = synth.f_shell(nk=4, nb=nb, nc=nc, nw=40, n_narrow=nc)
    e = wl.lattice.eps.reshape(4, nb)
    e[0, 1::2] = e[0, 0:2 * (nb // 2):2]
    e[0, 4] = e[0, 5] = e[0, 6]
    e[1, :12] = 0.3 + np.concatenate([[0.0], np.cumsum(10.0 ** np.arange(-13, -2, 1))])
    e[2, :] = -0.7
    e[3, :] = np.sort(e[3])[::-1]
    print("close energies", nb, nc, flush=True)
    check(ctx, wl, 0.1)


def test_non_orthonormal_rows_and_padded_orbitals(ctx):
    wl = synth.f_shell(nk=4, nb=37, nc=9, nw=30, n_narrow=9)
    rng = np.random.default_rng(2)
    m = np.eye(9) + 0.3 * (rng.standard_normal((9, 9)) + 1j * rng.standard_normal((9, 9))) / 3
    lat = synth.Lattice(4, 9, wl.lattice.nb, wl.lattice.eps, wl.lattice.wk,
                        np.concatenate([(m @ wl.lattice.proj_k(k)).ravel() for k in range(4)]))
    check(ctx, wl, -0.2, lat=lat)


def test_each_output_alone(ctx):
    """G_loc alone runs the kernel without the sums, N(k) or the scalars alone the
    one without the partials: the same bits as the full call."""
    from paper_1111_2157_amd.dyson import Lattice, SelfEnergy

    wl = synth.d_shell(nk=20, nb=33, nc=10, nw=50)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    nk, gl, sc = ctx.density_matrix(dl, ds, 0.25)
    only = [ctx.density_matrix(dl, ds, 0.25, nk=True, gloc=False, scalars=False)[0],
            ctx.gloc_compute(dl, ds, 0.25),
            ctx.density_matrix(dl, ds, 0.25, nk=False, gloc=False, scalars=True)[2]]
    ctx.sync_status()
    assert bool((only[0] == nk).all()) and bool((only[2] == sc).all())
    assert relerr(only[1].cpu().numpy(), gl.cpu().numpy()) < 1e-14


def test_sizes_on_different_kernels():
    """A ragged lattice whose 32-band windows run a low-rank and whose 64-band
    windows a dense kernel, the others the spectral one: the partials of the three
    add up."""
    from paper_1111_2157_amd.dyson import Context

    wl = synth.batched(nk=24, nb_lo=14, nb_hi=64, nw=24, n_iter=2)
    c = Context(0)
    c.set_variant(0, 32, [v for v in c.variants(0, 32) if v & 8 and v != SPEC][0])
    c.set_variant(0, 64, [v for v in c.variants(0, 64) if not v & 8][0])
    for s in range(2):
        mats, gl, sc = gpu_density(c, wl, 0.1, sig_index=s)
        assert_nk_parity(mats, wl.lattices[s], wl.sigmas[s], 0.1)
        assert_gloc_parity(gl, wl.lattices[s], wl.sigmas[s], 0.1)
    c.close()


@pytest.mark.parametrize("what", ["eps", "sigma", "proj"])
def test_non_finite_inputs_are_reported(ctx, what):
    from paper_1111_2157_amd._lib import DmftError
    from paper_1111_2157_amd.dyson import Lattice, SelfEnergy

    for value in (np.nan, np.inf):
        wl = synth.plain(nk=4, nb=20, nc=5, nw=20)
        a = {"eps": wl.lattice.eps, "sigma": wl.sigma.sigma, "proj": wl.lattice.proj}[what]
        if what == "eps" and np.isinf(value):
            continue  # 1 / (z - inf) = 0: a band that is not there
        a.reshape(-1)[7] = value
        print("non-finite", what, value, flush=True)
        ctx.density_matrix(Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma), 0.0)
        with pytest.raises(DmftError) as e:
            ctx.sync_status()
        assert e.value.name == "DMFT_ENONFINITE"
    check(ctx, synth.plain(nk=4, nb=20, nc=5, nw=20), 0.0)
