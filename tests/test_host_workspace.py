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


# the adjoint kinds' partials: 2.4 to 3 times these with k-tiles of their own choice; the
# sums of the spectral density pass are what remains
@pytest.mark.parametrize("nk,nb,nc,nw,size,more", [
    (8542, (13, 34), 1, 513, 2293073152, 1.0), (4111, 11, 10, 851, 1266592768, 1.3), (2294, 12, 7, 1252, 1263759616, 1.1)])
def test_adjoint_partials(lib, h, nk, nb, nc, nw, size, more):  # noqa: F811
    r, n = ws_size(lib, h, lattice(nk, nc, windows(nk, nb)), sigma(nw))
    assert r == 0 and n <= more * size, n / size


def test_one_size_serves_every_call(lib, h):  # noqa: F811
    """Over random shapes: with the size as asked for every kind of call reaches the device
    (which a planning handle does not have), with one byte less density_matrix does not."""
    rng = np.random.default_rng(5)
    out, ws = fake(200), fake(100)
    for i in range(60):
        nc = int(rng.integers(1, 17))
        nb = rng.integers(nc, rng.integers(nc, 65) + 1, int(2 ** rng.uniform(0, 12)))
        lat, sig = lattice(len(nb), nc, nb), sigma(int(2 ** rng.uniform(0, 11)))
        r, need = ws_size(lib, h, lat, sig)
        assert r == 0
        n = C.c_size_t(need)
        mu, passes, nv = C.c_double(), C.c_int(), C.c_double()
        assert lib.density_matrix(h, ref(lat), ref(sig), C.c_double(0.0), 2, out, None, None, ws, C.c_size_t(need - 1),
                                  None) == -6, (i, nc, len(nb), sig.nw)
        for r in (lib.density_matrix(h, ref(lat), ref(sig), C.c_double(0.0), 2, out, None, None, ws, n, None),
                  lib.dmft_ntot(h, ref(lat), ref(sig), C.c_double(0.0), 2, out, ws, n, None),
                  lib.dmft_ntot_vjp(h, ref(lat), ref(sig), C.c_double(0.0), 2, out, out, ws, n, None),
                  lib.density_matrix_vjp(h, ref(lat), ref(sig), C.c_double(0.0), 2, out, out, out, None, ws, n, None),
                  lib.find_mu(h, ref(lat), ref(sig), 2, C.c_double(1.0), C.c_double(1e-8), 0, C.c_double(-1.0),
                              C.c_double(1.0), C.c_double(0.0), 9, ref(mu), ref(passes), ref(nv), ws, n, None)):
            assert r == -1 and "planning handle" in last(lib, h), (i, nc, len(nb), sig.nw, last(lib, h))


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
