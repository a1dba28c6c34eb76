"""The autotuner checks its candidates against a dense code, which takes any projectors, and
against the error word: on a lattice with a dependent projector row a tuned handle gives
the oracle's numbers (1e-10 relative), whichever codes fail there, and a candidate's error
does not stay behind; one that was pending does."""
import numpy as np
import pytest

import oracle
from paper_1111_2157_amd import synth
from gpu_util import assert_gloc_parity, assert_nk_parity, gpu_density, relerr

pytestmark = pytest.mark.gpu


def dependent(nb, nc, nk=4, nw=21):
    wl = synth.f_shell(nk=nk, nb=nb, nc=nc, nw=nw, n_narrow=nc)
    p = wl.lattice.proj.reshape(nk, nc, nb)
    p[0, nc - 1] = p[0, 0]
    p[1, 1] = p[1, 0] + 1e-7 * p[1, 1]
    return wl


@pytest.mark.parametrize("nb,nc", [(12, 4), (30, 10), (40, 16), (50, 14)])
def test_tuned_on_dependent_rows(nb, nc):
    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = dependent(nb, nc)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    c = Context(0)
    try:
        print("autotune, dependent rows", nb, nc, flush=True)
        rep = c.autotune(dl, ds, 0.2)
        c.sync_status()  # nothing left behind by a rejected candidate
        nbp = (nb + 15) // 16 * 16
        for kind, name in enumerate(("density", "trace")):
            dense = [v for v in c.variants(kind, nbp) if not v & 8][0]
            assert any(name in x and "var=%d " % dense in x and "rejected" not in x for x in rep.splitlines()), rep
        mats, gl, _ = gpu_density(c, wl, 0.2)
        n = c.dmft_ntot(dl, ds, 0.2).cpu().numpy()
        c.sync_status()
        if nb <= 48:
            out, sb = c.dmft_ntot_vjp(dl, ds, 0.2)
            c.sync_status()
    finally:
        c.close()
    assert_nk_parity(mats, wl.lattice, wl.sigma, 0.2, 2)
    assert_gloc_parity(gl, wl.lattice, wl.sigma, 0.2)
    ref = oracle.trace(wl.lattice, wl.sigma, 0.2)
    got = [n] + ([out.cpu().numpy()] if nb <= 48 else [])
    for x in got:
        assert abs(x[0] - ref[0]) <= 1e-10 * abs(ref[0]) and abs(x[1] - ref[1]) <= 1e-10 * abs(ref[1])
    if nb <= 48:
        g, _ = oracle.vjp(wl.lattice, wl.sigma, 0.2, nbar=[wl.lattice.wk[k] * np.eye(nb) for k in range(4)])
        for j in range(wl.sigma.nw):
            assert relerr(sb[j].cpu().numpy(), g[j]) <= 1e-10, j


def test_pending_error_survives():
    from paper_1111_2157_amd._lib import DmftError
    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = synth.plain(nk=4, nb=12, nc=4, nw=16)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    bad = wl.sigma.sigma.copy()
    bad[3, 0, 0] = np.nan
    c = Context(0)
    try:
        c.autotune(dl, ds, 0.1)  # the workspace has its final size
        c.sync_status()
        print("pending error", flush=True)
        c.density_matrix(dl, SelfEnergy.from_host(synth.SelfEnergy(16, wl.sigma.beta, bad, wl.sigma.sigma_inf,
                                                                    wl.sigma.e_dc)), 0.1)
        c.autotune(dl, ds, 0.1)
        with pytest.raises(DmftError) as e:
            c.sync_status()
        assert e.value.name == "DMFT_ENONFINITE"
    finally:
        c.close()
