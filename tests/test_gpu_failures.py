"""Failed inversions: what is reported, and what they leave behind."""
import numpy as np
import pytest

from paper_0711_0999_amd import inputs

pytestmark = pytest.mark.gpu

KW = dict(U=1.0, E=1.5, n_eps=2, n_ebar=3, t_min=-1.0, t_max=2.0, dt=0.1, dtau=0.1, beta=1.3)


@pytest.mark.parametrize("bad", [np.nan, np.inf, complex(0.0, -np.inf)])
def test_failed_impurity_update_leaves_sigma(lib, bad):
    """The update runs to its end before the host sees that its inversion failed;
    later steps and norms are those of a context that has not failed."""
    print(f"case: impurity update with an entry {bad}", flush=True)
    good = inputs.random_sigma(73, seed=5, scale=0.1)
    broken = good.copy()
    broken[3, 17] = bad
    with lib.Context(**KW) as ctx, lib.Context(**KW) as fresh:
        ctx.set_sigma(good)
        ctx.compute_gloc()
        ctx.set_sigma(broken)
        with pytest.raises(lib.FkError, match="FK_ENONFINITE"):
            ctx.impurity_update()
        assert np.array_equal(ctx.get_sigma(), broken, equal_nan=True)
        with pytest.raises(lib.FkError, match="FK_ENONFINITE"):
            ctx.compute_gloc()
        with pytest.raises(lib.FkError, match="FK_ENONFINITE"):
            ctx.iterate(3)
        assert np.array_equal(ctx.get_sigma(), broken, equal_nan=True)
        results = []
        for c in (ctx, fresh):
            c.set_sigma(good)
            out = c.iterate(3)
            c.compute_gloc()
            resid = c.compute_gloc(lib.FK_MIXED)
            results.append((out, resid, c.impurity_update(), c.get_gloc(), c.get_sigma()))
        for a, b in zip(*results):
            np.testing.assert_equal(a, b)


STEP = 0.125


@pytest.mark.parametrize("n_c,n_ebar", [(99, 3), (300, 3), (600, 3), (1100, 3), (600, 12),
                                        (600, 25)])
def test_zero_pivot_is_named(lib, n_c, n_ebar):
    """The points at eps = 0 (the second of three nodes) hold an exactly singular
    2 x 2 block; without a field G0_k^-1 is exact there and the first of them is
    point n_ebar.  3 n_ebar matrices: split panels by groups and by quarters, and
    whole ones."""
    n_tau = 16 + n_c % 2
    n_t = (n_c - n_tau) // 2
    t_min = -STEP * (n_t // 4)
    with lib.Context(t_min=t_min, t_max=t_min + STEP * n_t, dt=STEP, dtau=STEP,
                     beta=STEP * n_tau, U=1.0, E=0.0, n_eps=3, n_ebar=n_ebar) as ctx:
        assert ctx.n_c == n_c
        i = np.arange(n_c)
        g0inv = np.zeros((n_c, n_c), complex)
        g0inv[i, i] = 1j
        g0inv[i[1:], i[1:] - 1] = -1j
        g0inv[0, n_c - 1] = 1j
        w = ctx.contour_points()[1]
        good = inputs.random_sigma(n_c, seed=n_c, scale=0.05)
        ctx.set_sigma(good)
        ctx.compute_gloc()
        first = ctx.get_gloc()
        ctx.set_refinement(0)
        for c in (5, 37, 70, n_c - 3):
            print(f"case: zero pivot at column {c + 1}, N_c = {n_c}, {3 * n_ebar} points",
                  flush=True)
            a = np.eye(n_c, dtype=complex)
            a[c, c + 1] = a[c + 1, c] = 1.0
            ctx.set_sigma((g0inv - a) / w[:, None] / w[None, :])
            for precision in (lib.FK_FP64, lib.FK_MIXED):
                with pytest.raises(lib.FkError, match="FK_ESINGULAR") as e:
                    ctx.compute_gloc(precision)
                assert f"zero pivot at column {c + 1} of matrix {n_ebar}" in str(e.value)
        ctx.set_sigma(good)
        ctx.compute_gloc()
        assert np.array_equal(ctx.get_gloc(), first)
