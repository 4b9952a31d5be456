"""The inversion's pivots, on point matrices made to order.

With one quadrature node in eps (0 exactly) and no field, G0_k^-1 has the exact
entries i (diagonal), -i (sub-diagonal) and i (corner); with steps of 1/8 the
weights are exact too, so Sigma = W^-1 (G0^-1 - A) W^-1 makes any chosen A of
short binary fractions the matrix that is inverted, for every ebar node."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STEP = 0.125


def made_to_order(lib, n_c, points=1):
    """A context of N_c = n_c and a function that maps A to its Sigma."""
    n_tau = 16 + n_c % 2
    n_t = (n_c - n_tau) // 2
    t_min = -STEP * (n_t // 4)
    ctx = lib.Context(t_min=t_min, t_max=t_min + STEP * n_t, dt=STEP, dtau=STEP,
                      beta=STEP * n_tau, U=1.0, E=0.0, n_eps=1, n_ebar=points)
    assert ctx.n_c == n_c

    def sigma(a):
        g0inv = np.zeros((n_c, n_c), complex)
        i = np.arange(n_c)
        g0inv[i, i] = 1j
        g0inv[i[1:], i[1:] - 1] = -1j
        g0inv[0, n_c - 1] = 1j
        w = ctx.contour_points()[1]
        return (g0inv - a) / w[:, None] / w[None, :]

    return ctx, sigma


@pytest.mark.parametrize("n_c", [100, 300, 600])
@pytest.mark.parametrize("power", [-60, -63, -66])
def test_small_pivots_in_complex64(lib, power, n_c):
    """Pivots whose squared modulus lies below the smallest normal float: their
    inverses are floats, and exact."""
    print(f"case: complex64 pivots 2^{power}, N_c = {n_c}", flush=True)
    ctx, sigma = made_to_order(lib, n_c)
    with ctx:
        a = np.zeros((n_c, n_c), complex)
        i = np.arange(n_c)
        a[i, (i + 1) % n_c] = 2.0 ** power
        ctx.set_sigma(sigma(a))
        ctx.set_refinement(0)
        ctx.compute_gloc(lib.FK_MIXED)
        expect = np.zeros((n_c, n_c), complex)
        expect[(i + 1) % n_c, i] = 2.0 ** -power
        assert np.array_equal(ctx.get_gloc(), expect)
