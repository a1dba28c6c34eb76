"""The spectral trace, scalar-adjoint and general-product kernels (variant 136, the
default of kinds 1 to 3) against the frequency-at-a-time low-rank kernels, which the
oracle tests cover: both ends of the padded sizes and orbital classes, frequency counts
around the group of 16, several k-points per work item, equal band energies, each
cotangent alone and neither.

Tolerance: both sides sum nk nw evaluations whose rounding error is about nc^2 2^-53
times the norms of two inverses, with condition numbers up to 1e3 here: 1e-10 of the
largest element, as for the variants against the oracle."""
import numpy as np
import pytest

from paper_1111_2157_amd import synth
from gpu_util import RTOL

pytestmark = pytest.mark.gpu

SPEC = 136


def _lattice(nk, nb, nc, nw, paired, ragged):
    rng = np.random.default_rng(100 * nb + nc)
    wl = synth.f_shell(nk=nk, nb=nb, nc=nc, nw=nw, n_narrow=min(nb, nc))
    lat = wl.lattice
    if paired:
        lat.eps[:] = np.round(lat.eps, 0)  # many equal energies in every window
    if ragged:
        nbs = rng.integers(max(nc, nb - 20), nb + 1, nk).astype(np.int32)
        eps = np.concatenate([wl.lattice.eps.reshape(nk, nb)[k, :m] for k, m in enumerate(nbs)])
        proj = np.concatenate([wl.lattice.proj.reshape(nk, nc, nb)[k, :, :m].reshape(-1) for k, m in enumerate(nbs)])
        lat = synth.Lattice(nk, nc, nbs, eps, lat.wk, np.ascontiguousarray(proj))
    return lat, wl.sigma


CASES = [(3, 1, 1, 1, 0, 0), (2, 16, 5, 17, 0, 0), (3, 17, 6, 15, 1, 0), (2, 32, 8, 33, 0, 0), (2, 33, 9, 16, 0, 0),
         (2, 48, 10, 31, 1, 0), (2, 49, 11, 18, 0, 0), (2, 64, 14, 20, 1, 0), (700, 6, 2, 20, 0, 0),
         (9, 60, 7, 40, 0, 1), (2500, 20, 13, 16, 0, 0)]


@pytest.mark.parametrize("nk,nb,nc,nw,paired,ragged", CASES)
def test_against_lowrank(nk, nb, nc, nw, paired, ragged):
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    lat, sig = _lattice(nk, nb, nc, nw, paired, ragged)
    dl, ds = Lattice.from_host(lat), SelfEnergy.from_host(sig)
    g = torch.Generator().manual_seed(nb)
    nbar = torch.randn(int((lat.nb.astype(np.int64) ** 2).sum()), generator=g, dtype=torch.complex128).cuda()
    gbar = torch.randn((nw, nc, nc), generator=g, dtype=torch.complex128).cuda()
    got = {}
    for form in ("spectral", "lowrank"):
        c = Context(0)
        try:
            for nbp in (16, 32, 48, 64):
                for kind in (1, 2, 3):
                    assert c.get_variant(kind, nbp) == SPEC
                    if form == "lowrank":
                        c.set_variant(kind, nbp, [v for v in c.variants(kind, nbp) if v & 8 and v != SPEC][0])
            print("spectral adj", form, nk, nb, nc, nw, flush=True)
            r = [c.dmft_ntot(dl, ds, 0.3), *c.dmft_ntot_vjp(dl, ds, 0.3)]
            for n_, g_ in ((nbar, gbar), (nbar, None), (None, gbar), (None, None)):
                r += c.density_matrix_vjp(dl, ds, 0.3, n_, g_)
            torch.cuda.synchronize()
            c.sync_status()
            got[form] = [x.cpu().numpy() for x in r]
        finally:
            c.close()
    for j, (x, y) in enumerate(zip(got["spectral"], got["lowrank"])):
        assert np.all(np.isfinite(x.view(np.float64))), j
        assert np.abs(x - y).max() <= RTOL * max(np.abs(y).max(), 1e-300), j
    assert not np.any(got["spectral"][-2])  # no cotangents: zero


def test_orbitals_past_the_widest_class(nk=2, nb=20, nc=16):
    """15 and 16 orbitals run the next variant of the list: the same numbers as when it is set."""
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = synth.f_shell(nk=nk, nb=nb, nc=nc, nw=12, n_narrow=nc)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    out = []
    for pin in (False, True):
        c = Context(0)
        try:
            if pin:
                for kind in (1, 2, 3):
                    c.set_variant(kind, 32, c.variants(kind, 32)[1])
            r = [c.dmft_ntot(dl, ds, 0.1), *c.dmft_ntot_vjp(dl, ds, 0.1)]
            torch.cuda.synchronize()
            c.sync_status()
            out.append([x.cpu().numpy() for x in r])
        finally:
            c.close()
    for x, y in zip(*out):
        assert np.abs(x - y).max() <= RTOL * np.abs(y).max()
