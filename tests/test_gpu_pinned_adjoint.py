"""A low-rank code set for the general product alone runs on its own default tiles: the
same sums, to the bit, as with the scalar adjoint set too (the two had shared a tile, taken
from the spectral form as soon as either ran it)."""
import pytest

from paper_1111_2157_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,nc", [(16, 12), (40, 5), (60, 14)])
def test_general_product_set_alone(nb, nc):
    import torch

    from paper_1111_2157_amd.dyson import Context, Lattice, SelfEnergy

    wl = synth.f_shell(nk=40, nb=nb, nc=nc, nw=100, n_narrow=nc)
    dl, ds = Lattice.from_host(wl.lattice), SelfEnergy.from_host(wl.sigma)
    g = torch.Generator().manual_seed(nb)
    nbar = torch.randn(40 * nb * nb, generator=g, dtype=torch.complex128).cuda()
    gbar = torch.randn((100, nc, nc), generator=g, dtype=torch.complex128).cuda()
    nbp = (nb + 15) // 16 * 16
    got = []
    for kinds in ((3,), (2, 3)):
        c = Context(0)
        try:
            for kind in kinds:
                c.set_variant(kind, nbp, [v for v in c.variants(kind, nbp) if v & 8 and v != 136][0])
            print("general product set alone", nb, nc, kinds, flush=True)
            got.append(c.density_matrix_vjp(dl, ds, 0.1, nbar, gbar))
            torch.cuda.synchronize()
            c.sync_status()
        finally:
            c.close()
    assert bool((got[0][0] == got[1][0]).all()) and bool((got[0][1] == got[1][1]).all())
