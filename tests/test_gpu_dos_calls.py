"""Calls of the DOS at the limits of what it takes: the largest finite
frequencies, more frequencies than one launch has threads for."""
import numpy as np
import pytest

from paper_0711_0999_amd import inputs

pytestmark = pytest.mark.gpu

KW = dict(U=1.0, E=1.5, n_eps=2, n_ebar=2, t_min=-0.4, t_max=2.4, dt=0.2, dtau=0.2, beta=1.2)


def test_largest_frequencies_at_the_ends_of_the_contour(lib):
    """Windows of D = 0 and 1 relative times: the phases w d h of later ones
    overflow, but no result depends on them.  With D = 6 they belong to the
    window, and the result is no number."""
    print("case: DOS at the largest finite frequencies", flush=True)
    big = np.finfo(float).max
    with lib.Context(**KW) as ctx:
        ctx.set_sigma(inputs.random_sigma(ctx.n_c, seed=3, scale=0.1))
        ctx.compute_gloc()
        g, n_t = ctx.get_gloc(), ctx.n_t
        for noalloc in (False, True):
            call = ctx.wigner_dos_noalloc if noalloc else ctx.wigner_dos
            rho = call([0, n_t - 1, 1], np.array([0.0, big, -big]))
            assert np.all(np.isfinite(rho))
            # D = 0: -(h / pi) Im f_0 / 2 at every frequency
            for r, i in ((0, 0), (1, n_t - 1)):
                f0 = g[2 * n_t - i, i] - g[i, 2 * n_t - i]
                assert np.allclose(rho[r], -0.4 / np.pi * 0.5 * f0.imag, rtol=1e-13, atol=0)
            rho = call([6], np.array([0.0, big, big / 4]))
            assert np.array_equal(np.isfinite(rho[0]), [True, False, True])


def test_more_frequencies_than_a_launch_has_threads_for(lib):
    """2^29 + 37 frequencies, eight threads each."""
    print("case: DOS at 2^29 + 37 frequencies", flush=True)
    n_w = 2 ** 29 + 37
    at = np.array([0, 1, 2 ** 28 - 1, 2 ** 28, 2 ** 29 - 1, 2 ** 29, n_w - 1])
    omega = np.zeros(n_w)
    omega[at] = 0.25 + np.arange(len(at))
    with lib.Context(**KW) as ctx:
        ctx.set_sigma(inputs.random_sigma(ctx.n_c, seed=3, scale=0.1))
        ctx.compute_gloc()
        rho = ctx.wigner_dos([5], omega)[0]
        few = ctx.wigner_dos([5], np.concatenate([omega[at], [0.0]]))[0]
    assert np.array_equal(rho[at], few[:-1])
    rho[at] = few[-1]
    assert np.all(rho == few[-1])
