"""DOS and PDOS kernel at the edges of its tiling: energies past a 32-energy block,
levels past a 256-level chunk and past a slice, one to sixteen orbitals, against the
same sums of the device's own eigensystem in float64.

Tolerance: every term is positive and is rounded a few times, and the longest chain of
additions is the number of levels, so the relative error stays below (levels + 16) 2^-52."""
import numpy as np
import pytest

from paper_1111_2157_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,nb,nc,ne", [(1, 1, 1, 1), (3, 16, 16, 31), (5, 9, 2, 33), (40, 13, 5, 64), (300, 8, 3, 97)])
def test_dos_against_sum(nk, nb, nc, ne):
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, PoleSelfEnergy

    rng = np.random.default_rng(nk + ne)
    eps = rng.uniform(-5.0, 5.0, nk * nb)
    x = rng.standard_normal((nk, nb, nc)) + 1j * rng.standard_normal((nk, nb, nc))
    proj = np.ascontiguousarray(np.linalg.qr(x)[0].conj().transpose(0, 2, 1))
    wk = rng.uniform(0.5, 1.5, nk) / nk
    lat = Lattice.from_host(synth.Lattice(nk, nc, np.full(nk, nb, np.int32), eps, wk, proj.reshape(-1)))
    v = torch.as_tensor(rng.standard_normal((2, nc)) + 1j * rng.standard_normal((2, nc)), device="cuda")
    pol = PoleSelfEnergy(2, 20.0, torch.tensor([-0.7, 1.3], dtype=torch.float64, device="cuda"), v,
                         torch.zeros((nc, nc), dtype=torch.complex128, device="cuda"),
                         torch.zeros(nc, dtype=torch.float64, device="cuda"))
    ctx = Context(0)
    try:
        print("pole dos", nk, nb, nc, ne, flush=True)
        es = ctx.pole_eig(lat, pol)
        dos, pdos = ctx.pole_dos(lat, pol, es, 0.25, 0.07, -6.0, 6.0, ne)
        ctx.sync_status()
    finally:
        ctx.close()
    lam = es.evals.cpu().numpy().reshape(nk, -1)
    w = wk[:, None] * es.wphys.cpu().numpy().reshape(lam.shape)
    wo = wk[:, None, None] * es.worb.cpu().numpy().reshape(lam.shape + (nc,))
    e = (np.linspace(-6.0, 6.0, ne) if ne > 1 else np.array([-6.0])) + 0.25
    lor = (0.07 / np.pi) / ((e[:, None, None] - lam[None]) ** 2 + 0.07 ** 2)
    # the argument e - lam loses a few ulps of e to its own rounding: amplified by at most |e| / eta
    tol = (lam.size + 16 + 4.0 * 7.0 / 0.07) * 2.0 ** -52
    np.testing.assert_allclose(dos.cpu().numpy(), (lor * w).sum((1, 2)), rtol=tol, atol=0)
    ref = np.einsum("ekl,kla->ea", lor, wo)
    # orbital weights may be zero: an absolute floor of their own rounding
    np.testing.assert_allclose(pdos.cpu().numpy(), ref, rtol=tol, atol=tol * np.abs(ref).max())
