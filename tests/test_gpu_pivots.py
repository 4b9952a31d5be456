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


def pairs(n_c, seed, gap=None):
    """Row pairs (r1[b], r2[b]), r1 < r2, of the 2 x 2 blocks on the columns 2b and
    2b + 1: random rows, or (gap) rows that lie `gap` apart."""
    rng = np.random.default_rng(seed)
    nb = n_c // 2
    if gap is None:
        r = rng.permutation(2 * nb).reshape(nb, 2)
        return r.min(1), r.max(1)
    free, r1, r2 = np.ones(n_c, bool), [], []
    for r in range(n_c - gap):
        if free[r] and free[r + gap]:
            free[r] = free[r + gap] = False
            r1.append(r)
            r2.append(r + gap)
    rest = np.flatnonzero(free)[: 2 * (nb - len(r1))].reshape(-1, 2)
    o = rng.permutation(nb)
    return (np.concatenate([r1, rest[:, 0]]).astype(int)[o],
            np.concatenate([r2, rest[:, 1]]).astype(int)[o])


def blocks(n_c, r1, r2, m, inv):
    """A with the 2 x 2 blocks m[b] in the rows (r1[b], r2[b]) and the columns
    (2b, 2b + 1), and its inverse from the blocks' inverses; a last odd row and
    column is completed by 1."""
    a, g = np.zeros((2, n_c, n_c), complex)
    for b, rows in enumerate(zip(r1, r2)):
        for p in range(2):
            for q in range(2):
                a[rows[p], 2 * b + q] = m[b, p, q]
                g[2 * b + q, rows[p]] = inv[b, q, p]
    if n_c % 2:
        r = np.setdiff1d(np.arange(n_c), np.concatenate([r1, r2]))[0]
        a[r, -1] = g[-1, r] = 1.0
    return a, g


def inverted(lib, n_c, points, a):
    """The inverse of A as a single point (FP64), and as G_loc in complex64 over
    the sum of the weights: both permuted copies of the stored inverse."""
    ctx, sigma = made_to_order(lib, n_c, points)
    with ctx:
        assert ctx.set_batch(points) == points
        ctx.set_sigma(sigma(a))
        ctx.compute_gloc()
        single = ctx.get_point_green(points // 2)
        ctx.set_refinement(0)
        ctx.compute_gloc(lib.FK_MIXED)
        return single, ctx.get_gloc() / ctx.points()[2].sum()


# rows: one form of the panel each (192, complex64 448, rows in LDS; one, two,
# four, six and more rows per thread); 1 and 33 matrices: split panels, 65: whole
FORMS = [(99, 1), (192, 1), (300, 1), (448, 1), (512, 1), (700, 1), (1025, 1), (2051, 1),
         (3073, 1), (700, 33), (300, 65), (700, 65), (1025, 65), (2051, 65), (3073, 65)]


@pytest.mark.parametrize("n_c,points", FORMS)
def test_largest_candidate_is_the_pivot(lib, n_c, points):
    """Candidates 1 and, in the higher row, p a little above it: with p as pivot
    the only rounding is that of 1 / p, while 1 as pivot leaves its remainder in
    the place of an exact zero.  Rows at random, one wave and one row slot apart."""
    for bits, gap in ((12, None), (12, 64), (12, 512), (18, None), (50, None)):
        if gap is not None and 2 * gap > n_c:
            continue
        print(f"case: candidates 2^-{bits} apart, gap {gap}, N_c = {n_c}, {points} points",
              flush=True)
        r1, r2 = pairs(n_c, n_c + bits, gap)
        nb = len(r1)
        p = 1 + 2.0 ** -bits
        f = np.float32(p)           # complex64: f = 1 ties with the lower row's 1
        m = np.tile(np.array([[1.0, 1.0], [p, 0.0]]), (nb, 1, 1))
        both = []
        for t in (p / (p * p), np.float64(f / (f * f))):
            inv = np.tile(np.array([[0.0, t], [1.0, -t]]), (nb, 1, 1))
            a, g = blocks(n_c, r1, r2, m, inv)
            both.append(g)
        single, mean = inverted(lib, n_c, points, a)
        assert np.array_equal(single, both[0])
        assert np.max(np.abs(mean - both[1])) < 1e-12


@pytest.mark.parametrize("n_c,points", FORMS)
def test_lowest_row_among_equal_candidates(lib, n_c, points):
    """Candidates 1 (the lower row) and 5/8 + 3/8 i of equal |re| + |im|: exact
    with the lower row as pivot, not with the other."""
    print(f"case: equal candidates, N_c = {n_c}, {points} points", flush=True)
    z = 0.625 + 0.375j
    for gap in (None, 64, 512):
        if gap is not None and 2 * gap > n_c:
            continue
        r1, r2 = pairs(n_c, n_c + 1, gap)
        nb = len(r1)
        m = np.tile(np.array([[1, 1], [z, z + 1]]), (nb, 1, 1))
        inv = np.tile(np.array([[z + 1, -1], [-z, 1]]), (nb, 1, 1))
        a, g = blocks(n_c, r1, r2, m, inv)
        single, mean = inverted(lib, n_c, points, a)
        assert np.array_equal(single, g)
        assert np.max(np.abs(mean - g)) < 1e-12
