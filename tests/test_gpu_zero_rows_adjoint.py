"""Correlated orbitals without weight in a k-point's window (zero projector rows) in the
adjoint passes and the batched pass, up to 16 orbitals and on either side of the default's
change of kernel, against the FP64 oracle: 1e-10 relative, as for every other input."""
import numpy as np
import pytest

import oracle
from paper_1111_2157_amd import synth
from gpu_util import assert_gloc_parity, assert_nk_parity, relerr

pytestmark = pytest.mark.gpu


def zero_rows(nb, nc, nk=4, nw=21):
    wl = synth.f_shell(nk=nk, nb=nb, nc=nc, nw=nw, n_narrow=min(nb, nc))
    proj = wl.lattice.proj.reshape(nk, nc, nb)
    proj[0, nc - 1] = 0.0
    proj[2, [0, nc // 2]] = 0.0
    proj[3] = 0.0
    return wl


def check_vjp(wl, codes=None):
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    lat, sig = wl.lattice, wl.sigma
    nk, nc, nb = lat.nk, lat.nc, int(lat.nb[0])
    g = torch.Generator().manual_seed(nb)
    nbar = torch.randn((nk, nb, nb), generator=g, dtype=torch.complex128)
    gbar = torch.randn((sig.nw, nc, nc), generator=g, dtype=torch.complex128)
    dl, ds = Lattice.from_host(lat), SelfEnergy.from_host(sig)
    c = Context(0)
    try:
        for kind, var in (codes or {}).items():
            c.set_variant(kind, (nb + 15) // 16 * 16, var)
        print("zero rows, adjoint", nb, nc, codes, flush=True)
        out, sb = c.dmft_ntot_vjp(dl, ds, 0.2)
        sg, mg = c.density_matrix_vjp(dl, ds, 0.2, nbar.reshape(-1).cuda(), gbar.cuda())
        torch.cuda.synchronize()
        c.sync_status()
    finally:
        c.close()
    n, d = oracle.trace(lat, sig, 0.2)
    o = out.cpu().numpy()
    assert abs(o[0] - n) <= 1e-10 * abs(n) and abs(o[1] - d) <= 1e-10 * max(abs(d), 1.0)
    r0, _ = oracle.vjp(lat, sig, 0.2, nbar=[lat.wk[k] * np.eye(nb) for k in range(nk)])
    r1, m1 = oracle.vjp(lat, sig, 0.2, nbar=[x.numpy() for x in nbar], gbar=gbar.numpy())
    for j in range(sig.nw):
        assert relerr(sb[j].cpu().numpy(), r0[j]) <= 1e-10, j
        assert relerr(sg[j].cpu().numpy(), r1[j]) <= 1e-10, j
    assert abs(float(mg[0]) - m1) <= 1e-10 * max(abs(m1), float(torch.linalg.vector_norm(nbar)))


@pytest.mark.parametrize("nb,nc", [(9, 3), (20, 5), (30, 10), (12, 12), (16, 14), (50, 14), (16, 16), (20, 15), (40, 16),
                                   (64, 15)])
def test_default_codes(nb, nc):
    check_vjp(zero_rows(nb, nc))


@pytest.mark.parametrize("nb,nc", [(12, 4), (16, 12), (40, 7), (60, 14)])
def test_low_rank_codes(nb, nc):
    """Set, whatever the default is; every code of the two kinds."""
    from paper_1111_2157_amd.dyson import Context

    c = Context(0)
    lists = [[v for v in c.variants(kind, (nb + 15) // 16 * 16) if v & 8 and v != 136] for kind in (2, 3)]
    c.close()
    for i in range(max(len(x) for x in lists)):
        check_vjp(zero_rows(nb, nc), {2: lists[0][i % len(lists[0])], 3: lists[1][i % len(lists[1])]})


@pytest.mark.parametrize("nc,nk,nw", [(14, 700, 16), (14, 701, 5), (11, 30, 40)])
def test_either_side_of_the_small_call_rule(nc, nk, nw):
    """16-band windows with 11 to 14 orbitals: the general product's kernel goes by the number
    of groups of 16 frequencies over all k-points (700; up to 12 orbitals it is one)."""
    check_vjp(zero_rows(16, nc, nk, nw))


def test_batched_pass():
    import torch

    from paper_1111_2157_amd.dyson import FORM_LOWRANK, Context, Lattice, SelfEnergy, split_nk

    wls = [zero_rows(24, 5), zero_rows(24, 16)]
    c = Context(0)
    try:
        c.batched_set_form(FORM_LOWRANK)
        lats = [Lattice.from_host(w.lattice) for w in wls]
        print("zero rows, batched", flush=True)
        c.batched_plan(lats, [SelfEnergy.from_host(w.sigma) for w in wls], 2)
        nks, gls = c.batched_outputs()
        c.batched_pass(torch.tensor([0.1, -0.2], dtype=torch.float64, device="cuda"), nks, gls)
        c.batched_sync_status()
        for s, mu in ((0, 0.1), (1, -0.2)):
            mats = [m.cpu().numpy() for m in split_nk(nks[s], lats[s])]
            assert_nk_parity(mats, wls[s].lattice, wls[s].sigma, mu, 2)
            assert_gloc_parity(gls[s].cpu().numpy(), wls[s].lattice, wls[s].sigma, mu)
    finally:
        c.close()
