"""Rounding error of the gradient in double against 64-bit mantissas (numpy's
long double) on the same inputs: no larger than that of the plain evaluation,
where every product of the staple is summed by itself before it is added and
the commutators of the series are formed term by term. Its rms over the
lattice, measured with the same inputs, is given per case; 1 % more is allowed,
the scatter of an rms over 9216 components.

The reference takes the derivative of exp from the exponential of a block
matrix: exp([[S, X], [0, S]]) has d exp(S)[X] as its upper right block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIMS = (6, 4, 6, 8)  # nx, ny, nz, nt
# (gauge, storage form, amplitude of s): rms of the error over rms of the gradient
REFERENCE = {(0, 0, 0.1): 2.8079e-16, (0, 1, 0.1): 3.8837e-16, (0, 0, 1.0): 6.0075e-16, (0, 1, 1.0): 6.4254e-16,
             (1, 0, 0.1): 2.7588e-16, (1, 1, 0.1): 3.8218e-16, (1, 0, 1.0): 5.9531e-16, (1, 1, 1.0): 6.4683e-16}


def generators():
    l = np.zeros((8, 3, 3), dtype=np.clongdouble)
    l[0][0, 1] = l[0][1, 0] = 1
    l[1][0, 1], l[1][1, 0] = -1j, 1j
    l[2][0, 0], l[2][1, 1] = 1, -1
    l[3][0, 2] = l[3][2, 0] = 1
    l[4][0, 2], l[4][2, 0] = -1j, 1j
    l[5][1, 2] = l[5][2, 1] = 1
    l[6][1, 2], l[6][2, 1] = -1j, 1j
    r3 = 1 / np.sqrt(np.longdouble(3))
    l[7][0, 0] = l[7][1, 1] = r3
    l[7][2, 2] = -2 * r3
    return 0.5j * l


def inputs(amp):
    rng = np.random.default_rng(5)
    shape = DIMS[::-1]
    z = rng.standard_normal(shape + (4, 3, 3)) + 1j * rng.standard_normal(shape + (4, 3, 3))
    q, _ = np.linalg.qr(z)
    U = q / np.linalg.det(q)[..., None, None] ** (1 / 3)
    return U, amp * rng.standard_normal(shape + (8,))


def mul(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def expm(x):
    y, e = x / 1024, np.broadcast_to(np.eye(x.shape[-1], dtype=x.dtype), x.shape)
    one = e
    for k in range(9, 0, -1):
        e = one + mul(y, e) / k
    for _ in range(10):
        e = mul(e, e)
    return e


def exact(U, s, nd):
    U, X = U.astype(np.clongdouble), generators()
    S = (s.astype(np.longdouble)[..., None, None] * X).sum(-3)
    dag = lambda a: a.conj().swapaxes(-1, -2)
    B = np.zeros(s.shape + (6, 6), dtype=np.clongdouble)
    B[..., :3, :3] = B[..., 3:, 3:] = S[..., None, :, :]
    B[..., :3, 3:] = X
    B = expm(B)
    g, dg = B[..., 0, :3, :3], B[..., :3, 3:]
    K = 0
    for mu in range(nd):
        ax = 3 - mu
        K = K + mul(U[..., mu, :, :], dag(np.roll(g, -1, ax)))
        K = K + mul(dag(np.roll(U[..., mu, :, :], 1, ax)), dag(np.roll(g, 1, ax)))
    d = (dg * K.swapaxes(-1, -2)[..., None, :, :]).sum((-1, -2)).real  # Re Tr dg_a K
    return d / (nd * 3 * np.prod(DIMS))


@pytest.mark.parametrize("gauge,store,amp", REFERENCE)
def test_error_is_no_larger_than_that_of_products_summed_apart(gauge, store, amp):
    import torch
    from paper_1412_1498_amd import gf
    U, s = inputs(amp)
    ctx = gf.Context(DIMS, gauge=gauge, prec=gf.F64, params=gf.default_params(gf.F64, storage=store))
    got = ctx.unpack_alg(ctx.functional_grad(ctx.pack(torch.from_numpy(U).cuda()),
                                             ctx.pack_alg(torch.from_numpy(s).cuda()))).cpu().numpy()
    want = exact(U, s, 4 if gauge == 0 else 3)
    rms = float(np.sqrt(((got - want) ** 2).mean() / (want ** 2).mean()))
    print(gauge, store, amp, rms)
    assert rms <= 1.01 * REFERENCE[gauge, store, amp]
