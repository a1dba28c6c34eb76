"""CPU tests of the workspace size through a planning handle: it holds whatever kernel
variants are chosen after it was asked for, without adding up the partials of both forms
of the density pass."""
import ctypes as C

import numpy as np
import pytest

from test_host_planning import fake, h, last, lattice, lib, ref, sigma, ws_size  # noqa: F401  (h, lib: fixtures)


def windows(nk, nb):
    if np.isscalar(nb):
        return np.full(nk, nb, np.int32)
    return np.random.default_rng(1).integers(nb[0], nb[1] + 1, nk).astype(np.int32)


# bytes with the partials of the band-window kernels alone
@pytest.mark.parametrize("nk,nb,nc,nw,size", [
    (64, 12, 5, 256, 84605184), (123, 27, 7, 333, 237722112), (512, 48, 14, 2048, 1694211584),
    (20000, 48, 14, 512, 7696360448), (4096, (20, 64), 5, 2048, 6490818048), (4096, (20, 64), 14, 2048, 6504826368)])
def test_one_form_at_a_time(lib, h, nk, nb, nc, nw, size):  # noqa: F811
    lat = lattice(nk, nc, windows(nk, nb))
    if np.isscalar(nb):
        lat.nb = None
    r, n = ws_size(lib, h, lat, sigma(nw))
    assert r == 0, last(lib, h)
    # windows of several sizes may be in either form each; there the spectral form's
    # partials are the larger ones for some
    assert n <= size * (1.0 if np.isscalar(nb) else 1.1)


@pytest.mark.parametrize("nk,nb,nc,nw", [(64, 12, 5, 256), (40, (8, 64), 6, 100), (200, (14, 64), 14, 64), (3, 64, 16, 40)])
def test_holds_any_choice_of_variants(lib, h, nk, nb, nc, nw):  # noqa: F811
    """density_matrix with the size as asked for at first reaches the device (which a planning
    handle does not have), whatever is set for each padded size."""
    lat, sig = lattice(nk, nc, windows(nk, nb)), sigma(nw)
    r, need = ws_size(lib, h, lat, sig)
    assert r == 0
    buf = (C.c_int * 16)()
    for choice in range(16):
        for i, nbp in enumerate((16, 32, 48, 64)):
            codes = buf[:lib.dmft_variants(0, nbp, buf, 16)]
            assert lib.dmft_set_variant(h, 0, nbp, 136 if choice >> i & 1 else [v for v in codes if not v & 8][0]) == 0
        assert ws_size(lib, h, lat, sig) == (0, need), choice
        assert lib.density_matrix(h, ref(lat), ref(sig), C.c_double(0.0), 2, fake(200), None, None, fake(100),
                                  C.c_size_t(need), None) == -1
        assert "planning handle" in last(lib, h)
