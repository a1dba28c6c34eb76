"""The one-matrix-per-lane form of the spectral density kernel (up to five orbitals)
around its groups of 64 frequencies, against the FP64 oracle: 1e-10 relative,
normwise per k and per frequency, as for the other variants."""
import pytest

from paper_1111_2157_amd import synth
from gpu_util import assert_gloc_parity, assert_nk_parity, gpu_density

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [63, 65, 130])
@pytest.mark.parametrize("nb,nc", [(13, 2), (16, 5), (31, 5), (64, 3), (64, 5)])
def test_groups_of_64(nw, nb, nc):
    from paper_1111_2157_amd.dyson import Context

    wl = synth.plain(nk=3, nb=nb, nc=nc, nw=nw)
    c = Context(0)
    try:
        print("lane", nb, nc, nw, flush=True)
        mats, gl, _ = gpu_density(c, wl, 0.2)
    finally:
        c.close()
    assert_nk_parity(mats, wl.lattice, wl.sigma, 0.2, 2)
    assert_gloc_parity(gl, wl.lattice, wl.sigma, 0.2)
