"""Contours whose sizes sit at the edges of the inversion's tiles, against the
oracle: row and column tiles of 64 with 1, 16, 17 or 63 left over, and a last
chunk of K (16 columns) that is whole, nearly empty or nearly full.

Bars: FP64 1e-10 of the largest value, as for every lattice step; one FP64
refinement step of the complex64 inverse 1e-8 (its products run through the
same tiles)."""
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


def lattice(kw, sig, n_eps, n_ebar):
    p = dmft.Problem(u=1.0, e_field=1.5, n_eps=n_eps, n_ebar=n_ebar, **kw)
    return dmft.lattice_only(p, sig)[:2]


@pytest.mark.parametrize("n_c", [64, 65, 80, 81, 127, 128, 129, 144, 335])
def test_tile_and_chunk_edges(lib, n_c):
    print(f"case: N_c = {n_c}, FP64 and refined complex64", flush=True)
    kw = contour(n_c)
    with lib.Context(U=1.0, E=1.5, n_eps=2, n_ebar=3, **kw) as ctx:
        assert ctx.n_c == n_c
        sig = inputs.random_sigma(n_c, seed=n_c, scale=0.2)
        go, jo = lattice(kw, sig, 2, 3)
        ctx.set_sigma(sig)
        ctx.compute_gloc()
        assert relerr(ctx.get_gloc(), go) < 1e-10
        assert relerr(ctx.get_current()[1], jo) < 1e-10
        ctx.set_refinement(1)
        ctx.compute_gloc(lib.FK_MIXED)
        assert relerr(ctx.get_gloc(), go) < 1e-8


# rows left of a block pick the panel's form: 192 (448 in complex64) rows in
# LDS, 512, 1024, 2048, 3072 and more rows in registers; the first block of
# n_c rows sits on each side of a line, the later ones cross the ones below
@pytest.mark.parametrize("n_c", [1, 0, -1])
@pytest.mark.parametrize("line", [192, 448, 512, 1024, 2048])
def test_panel_forms(lib, line, n_c):
    n_c += line
    print(f"case: N_c = {n_c}, panel line {line}", flush=True)
    kw = contour(n_c)
    with lib.Context(U=1.0, E=1.5, n_eps=1, n_ebar=2, **kw) as ctx:
        assert ctx.n_c == n_c
        sig = inputs.random_sigma(n_c, seed=n_c, scale=0.1)
        go, jo = lattice(kw, sig, 1, 2)
        ctx.set_sigma(sig)
        ctx.compute_gloc()
        assert relerr(ctx.get_gloc(), go) < 1e-10
        assert relerr(ctx.get_current()[1], jo) < 1e-10
        ctx.set_refinement(1)
        ctx.compute_gloc(lib.FK_MIXED)
        assert relerr(ctx.get_gloc(), go) < 1e-8


def test_equal_pivot_candidates(lib):
    """Sigma = 0 leaves columns whose candidates have equal magnitude: the
    lowest row wins, in every run the same."""
    print("case: equal pivot candidates, Sigma = 0", flush=True)
    kw = contour(259)
    with lib.Context(U=1.0, E=0.0, n_eps=3, n_ebar=3, **kw) as ctx:
        first = None
        for _ in range(2):
            ctx.set_sigma(np.zeros((259, 259), complex))
            ctx.compute_gloc()
            g = ctx.get_gloc()
            first = g if first is None else first
        assert np.array_equal(first, g)
    p = dmft.Problem(u=1.0, e_field=0.0, n_eps=3, n_ebar=3, **kw)
    go = dmft.lattice_only(p, np.zeros((259, 259), complex))[0]
    assert relerr(g, go) < 1e-10


@pytest.mark.parametrize("n_c", [193, 449, 513, 1025, 2049])
def test_split_panels_equal_whole_ones(lib, n_c):
    """65 matrices in one batch factor each block in one launch, batches of 13
    in several: the same steps, so G_loc differs by the order of its sum only."""
    print(f"case: N_c = {n_c}, whole and split panels", flush=True)
    kw = contour(n_c)
    with lib.Context(U=1.0, E=1.5, n_eps=5, n_ebar=13, **kw) as ctx:
        ctx.set_sigma(inputs.random_sigma(n_c, seed=n_c, scale=0.1))
        ctx.set_refinement(0)
        for precision, bar in ((lib.FK_FP64, 1e-12), (lib.FK_MIXED, 1e-6)):
            got = []
            for batch in (65, 13):
                assert ctx.set_batch(batch) == batch
                ctx.compute_gloc(precision)
                got.append(ctx.get_gloc())
            assert relerr(got[1], got[0]) < bar


def test_split_panels_of_many_rows_equal_whole_ones(lib):
    """The largest rows-per-thread form, whose split panels are launches per
    group of columns."""
    test_split_panels_equal_whole_ones(lib, 3073)


def test_split_panels_of_uneven_matrices(lib):
    """A few uneven matrices in one batch: small ones end inside a quarter and
    inside a group of columns of a panel that the largest one splits by groups."""
    sizes = (1155, 140, 170, 129)
    print(f"case: uneven split panels, N_c = {sizes}", flush=True)
    inst = [dict(U=1.0, E=1.5, n_eps=1, n_ebar=2, **contour(n)) for n in sizes]
    sig = [inputs.random_sigma(n, seed=n, scale=0.1) for n in sizes]
    with lib.Batch(inst) as b:
        for i, s in enumerate(sig):
            b.instance(i).set_sigma(s)
        b.iterate(1, 0.0)
        for i, n in enumerate(sizes):
            go, jo = lattice(contour(n), sig[i], 1, 2)
            assert relerr(b.instance(i).get_gloc(), go) < 1e-10
            assert relerr(b.instance(i).get_current()[1], jo) < 1e-10
