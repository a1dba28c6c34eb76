"""A handle tuned at one orbital count and used at another, and one whose variant is set
after tuning: the measured tile goes with the kernel it was measured on."""
import pytest

import oracle
from paper_1111_2157_amd import synth
from gpu_util import assert_gloc_parity, assert_nk_parity, gpu_density

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,then", [(5, 14), (14, 5), (10, 8)])
def test_tuned_then_other_orbitals(first, then):
    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wls = {nc: synth.f_shell(nk=64, nb=40, nc=nc, nw=200, n_narrow=nc) for nc in (first, then)}
    dev = {nc: (Lattice.from_host(w.lattice), SelfEnergy.from_host(w.sigma)) for nc, w in wls.items()}
    c, fresh = Context(0), Context(0)
    try:
        print("tuned at", first, "used at", then, flush=True)
        c.autotune(*dev[first], 0.1)
        c.sync_status()
        for kind in range(3):  # the codes chosen at the first count are not what is looked at here
            c.set_variant(kind, 48, -1)
        assert c.workspace_size(*dev[then]) == fresh.workspace_size(*dev[then])
        mats, gl, _ = gpu_density(c, wls[then], 0.1)
        n = c.dmft_ntot(*dev[then], 0.1).cpu().numpy()
        c.sync_status()
    finally:
        c.close()
        fresh.close()
    assert_nk_parity(mats, wls[then].lattice, wls[then].sigma, 0.1, 2, klist=[0, 31, 63])
    assert_gloc_parity(gl, wls[then].lattice, wls[then].sigma, 0.1, nlist=[0, 1, 63, 64, 199])
    ref = oracle.trace(wls[then].lattice, wls[then].sigma, 0.1)
    assert abs(n[0] - ref[0]) <= 1e-10 * abs(ref[0])


def test_variant_set_after_tuning():
    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = synth.f_shell(nk=64, nb=40, nc=14, nw=200, n_narrow=14)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    c, fresh = Context(0), Context(0)
    try:
        c.autotune(dl, ds, 0.1)
        c.sync_status()
        assert c.get_variant(0, 48) == 136
        for v in c.variants(0, 48)[1:3]:
            for x in (c, fresh):
                x.set_variant(0, 48, v)
            print("set after tuning", v, flush=True)
            a, b = (gpu_density(x, wl, 0.1) for x in (c, fresh))
            assert (a[1] == b[1]).all() and (a[2] == b[2]).all()  # the same tiles, so the same sums
    finally:
        c.close()
        fresh.close()
    assert_nk_parity(a[0], wl.lattice, wl.sigma, 0.1, 2, klist=[0, 31, 63])
    assert_gloc_parity(a[1], wl.lattice, wl.sigma, 0.1, nlist=[0, 1, 63, 64, 199])
