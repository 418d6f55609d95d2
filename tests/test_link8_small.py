"""8-real links with elements far below the rounding of the others: the phase
code of U00 and U20 (tests/test_link8.py) holds down to moduli whose squares
are the smallest normal doubles, and below, where the squares are subnormal,
as far as these resolve the modulus. A modulus whose square underflows to 0 is
coded as the number 0, as an exact 0 is."""
import cmath

import numpy as np
import pytest

U64 = 2.0 ** -53
MODULI = [1e-8, 1e-100, 1e-149, 1e-151, 1e-152, 1e-153, 1e-155, 1e-158]
ANGLES = [0.0, 0.4, 1.3, np.pi / 2, 2.2, -0.9, -2.9]


def link(m, ang):
    """An SU(3) matrix with U00 and U20 of modulus m (to rounding) and phases ang and -ang / 2."""
    a, c = m * cmath.exp(1j * ang), m * cmath.exp(-0.5j * ang)
    return np.array([[a, 0, 1], [1, 0, -a.conjugate()], [c, 1, 0]], dtype=complex)


def decode_phase(p):
    if abs(p) > 3:
        return 0j
    neg = abs(p) > 1
    t = np.copysign(2 - abs(p), p) if neg else p
    c = (1 - t * t) / (1 + t * t)
    return complex(-c if neg else c, 2 * t / (1 + t * t))


def tolerance(m):
    """8 units of roundoff as for ordinary elements; of a subnormal square three
    roundings by half the smallest number, 2^-1075 each (a product, the sum, the
    root's residual), halved by the root; the phase changes by no more than the
    modulus does. 2^-1074 in all."""
    return 8 * U64 + 2.0 ** -1074 / m ** 2


def check(stored, U, m):
    for k, z in ((6, U[0, 0]), (7, U[2, 0])):
        # |z| by scaling: both parts times 2^500 are ordinary numbers
        w = complex(z.real * 2.0 ** 500, z.imag * 2.0 ** 500)
        assert abs(decode_phase(stored[k]) - w / abs(w)) <= tolerance(m), (k, z, stored[k])


@pytest.mark.parametrize("m", MODULI)
@pytest.mark.parametrize("ang", ANGLES)
def test_phase_codes_of_small_elements(m, ang):
    from paper_1412_1498_amd import gf
    U = link(m, ang)
    stored, _ = gf.host_link8(0, U)
    check(stored, U, m)


def test_underflowing_elements_are_coded_as_zero():
    from paper_1412_1498_amd import gf
    for m in (0.0, 1e-163, 1e-200, 1e-320):
        stored, _ = gf.host_link8(0, link(m, 0.7))
        assert stored[6] == 4 and stored[7] == 4


@pytest.mark.gpu
def test_phase_codes_of_small_elements_on_the_gpu():
    import torch
    from paper_1412_1498_amd import gf
    dims = (4, 4, 2, 2)
    ctx = gf.Context(dims, prec=gf.F64, params=gf.default_params(gf.F64, storage=gf.STORE_8))
    cases = [(m, a) for m in MODULI for a in ANGLES]
    A = np.stack([link(*cases[i % len(cases)]) for i in range(4 * 64)]).reshape(2, 2, 4, 4, 4, 3, 3)
    S = ctx.pack(torch.from_numpy(A).cuda()).cpu().numpy()  # [parity][block][mu][element][site in block][re, im]
    for n in range(64):
        x, y, z, t = n % 4, n // 4 % 4, n // 16 % 2, n // 32
        for mu in range(4):
            m, a = cases[(4 * n + mu) % len(cases)]
            e = S[(x + y + z + t) % 2, 0, mu, :, n // 2]
            check(e.reshape(-1), link(m, a), m)
