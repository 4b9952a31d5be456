"""The panel's schedules against each other, point by point, and the one of 33 to
64 matrices against the oracle.  Forms by the rows left and the batch: up to 32
matrices with 513 to 1024 rows split by groups of columns, 33 to 64 by quarters,
more than 64 in one launch.

The schedules take the same steps on the same numbers, so a point's inverse is the
same bit for bit.  Bars against the oracle: those of every lattice step (FP64
1e-10, one refinement step 1e-8, complex64 1e-4)."""
import numpy as np
import pytest

from oracle import dmft
from paper_0711_0999_amd import inputs

pytestmark = pytest.mark.gpu


def contour(n_c):
    n_tau = 20 + n_c % 2
    n_t = (n_c - n_tau) // 2
    t_min = -0.1 * (n_t // 4)
    return dict(t_min=t_min, t_max=t_min + 0.1 * n_t, dt=0.1, dtau=0.1, beta=0.1 * n_tau)


def relerr(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("n_c", [193, 449, 513, 600, 1025, 2049])
def test_points_are_the_same_in_every_schedule(lib, n_c):
    print(f"case: N_c = {n_c}, batches of 65, 33 and 13", flush=True)
    with lib.Context(U=1.0, E=1.5, n_eps=5, n_ebar=13, **contour(n_c)) as ctx:
        ctx.set_sigma(inputs.random_sigma(n_c, seed=n_c, scale=0.1))
        ctx.set_refinement(0)
        want, low = {}, []
        for batch in (65, 33, 13):
            assert ctx.set_batch(batch) == batch
            ctx.compute_gloc()
            for k in (52, 57, 64):
                g = ctx.get_point_green(k)
                assert np.array_equal(g, want.setdefault(k, g)), (batch, k)
            ctx.compute_gloc(lib.FK_MIXED)
            low.append(ctx.get_gloc())
        # complex64 keeps no points: the same sums in another order, in FP64
        assert relerr(low[1], low[0]) < 1e-12 and relerr(low[2], low[0]) < 1e-12


@pytest.mark.parametrize("n_c", [513, 600, 1025])
def test_33_matrices_against_the_oracle(lib, n_c):
    print(f"case: N_c = {n_c}, 33 matrices", flush=True)
    kw = contour(n_c)
    sig = inputs.random_sigma(n_c, seed=n_c, scale=0.1)
    p = dmft.Problem(u=1.0, e_field=1.5, n_eps=3, n_ebar=11, **kw)
    go, jo = dmft.lattice_only(p, sig)[:2]
    with lib.Context(U=1.0, E=1.5, n_eps=3, n_ebar=11, **kw) as ctx:
        assert ctx.set_batch(33) == 33
        ctx.set_sigma(sig)
        ctx.compute_gloc()
        assert relerr(ctx.get_gloc(), go) < 1e-10
        assert relerr(ctx.get_current()[1], jo) < 1e-10
        for steps, bar in ((1, 1e-8), (0, 1e-4)):
            ctx.set_refinement(steps)
            ctx.compute_gloc(lib.FK_MIXED)
            assert relerr(ctx.get_gloc(), go) < bar
            assert relerr(ctx.get_current()[1], jo) < bar


@pytest.mark.parametrize("n_c", [330, 600, 1100, 2200])
def test_second_stream_and_tile_heights_change_nothing(lib, n_c):
    """Split panels on the second stream beside the trailing updates, both tile
    heights: every element takes the same sums."""
    print(f"case: N_c = {n_c}, look-ahead and tiles of 128 rows", flush=True)
    with lib.Context(U=1.0, E=1.5, n_eps=2, n_ebar=3, **contour(n_c)) as ctx:
        ctx.set_sigma(inputs.random_sigma(n_c, seed=n_c, scale=0.1))
        ctx.set_refinement(0)
        want = None
        for rows in (64, 128):
            for ahead in (0, 1, 1):
                ctx.set_tuning(tile_rows=rows, batch=6, lookahead=ahead)
                ctx.compute_gloc()
                got = [ctx.get_point_green(k) for k in (0, 5)]
                ctx.compute_gloc(lib.FK_MIXED)
                got.append(ctx.get_gloc())
                want = want or got
                assert all(np.array_equal(a, b) for a, b in zip(got, want)), (rows, ahead)
