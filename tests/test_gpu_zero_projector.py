"""Correlated orbitals without weight in a k-point's band window (zero projector rows):
the default density, trace and adjoint passes against the FP64 oracle, which inverts the
band-window matrix.  1e-10 relative, as for every other input."""
import numpy as np
import pytest

import oracle
from paper_1111_2157_amd import synth
from gpu_util import assert_gloc_parity, assert_nk_parity, gpu_density, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,nc", [(9, 3), (20, 5), (40, 5), (18, 7), (30, 10), (50, 14)])
def test_zero_projector_rows(nb, nc):
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = synth.f_shell(nk=4, nb=nb, nc=nc, nw=21, n_narrow=nc)
    proj = wl.lattice.proj.reshape(4, nc, nb)
    proj[0, nc - 1] = 0.0          # one orbital at one k-point
    proj[2, [0, nc // 2]] = 0.0    # two at another
    proj[3] = 0.0                  # all of them
    c = Context(0)
    try:
        print("zero rows", nb, nc, flush=True)
        mats, gl, _ = gpu_density(c, wl, 0.2)
        dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
        n1 = c.dmft_ntot(dl, ds, 0.2).cpu().numpy()
        out, sb = c.dmft_ntot_vjp(dl, ds, 0.2)
        torch.cuda.synchronize()
        c.sync_status()
    finally:
        c.close()
    assert_nk_parity(mats, wl.lattice, wl.sigma, 0.2, 2)
    assert_gloc_parity(gl, wl.lattice, wl.sigma, 0.2)
    n, d = oracle.trace(wl.lattice, wl.sigma, 0.2)
    for got in (n1, out.cpu().numpy()):
        assert abs(got[0] - n) <= 1e-10 * abs(n) and abs(got[1] - d) <= 1e-10 * abs(d)
    ref, _ = oracle.vjp(wl.lattice, wl.sigma, 0.2, nbar=[wl.lattice.wk[k] * np.eye(nb) for k in range(4)])
    for j in range(wl.sigma.nw):
        assert relerr(sb[j].cpu().numpy(), ref[j]) <= 1e-10, j
