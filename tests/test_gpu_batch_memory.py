"""Device memory of a sweep that is cut into many small chunks, and its results."""
import numpy as np
import pytest

from paper_0711_0999_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")   # before the library initializes the device


def contour(n_c):
    n_tau = 20 + n_c % 2
    n_t = (n_c - n_tau) // 2
    t_min = -0.1 * (n_t // 4)
    return dict(t_min=t_min, t_max=t_min + 0.1 * n_t, dt=0.1, dtau=0.1, beta=0.1 * n_tau)


def per_matrix(n):
    """Bytes of a chunk's matrix: itself and 512 gathered rows, the pivots."""
    return 16.0 * (n * n + 512 * n) + 8.0 * n


def test_small_chunks_share_their_buffers(lib):
    """16 instances of 256 points, N_c = 200, in 64 chunks of 64 matrices: 147 MB
    of chunk storage and 37 MB of impurity slots, whatever the number of chunks;
    a buffer of 16 MiB of each chunk's own would be another 1074 MB."""
    print("case: memory of 64 chunks", flush=True)
    kw = dict(U=1.0, E=1.5, n_eps=16, n_ebar=16, **contour(200))
    torch.zeros(1, device="cuda")
    with lib.Batch([kw] * 16) as b:
        free = torch.cuda.mem_get_info()[0]
        b.set_chunk_bytes(64.5 * per_matrix(200))
        b.iterate(1, 0.0)
        assert free - torch.cuda.mem_get_info()[0] < 600e6


@pytest.mark.parametrize("chunk", [1, 7, 40])
def test_chunks_of_any_size_agree(lib, chunk):
    """Uneven instances, split panels in every chunk and in the impurity update
    after them, against one chunk of all the matrices."""
    sizes = (210, 560, 97, 330)
    print(f"case: sweep in chunks of {chunk} of the largest matrices", flush=True)
    kws = [dict(U=1.0, E=1.5, n_eps=4, n_ebar=5, **contour(n)) for n in sizes]
    sig = [inputs.random_sigma(n, seed=n, scale=0.1) for n in sizes]
    got = []
    for size in (1e12, (chunk + 0.5) * per_matrix(560)):
        with lib.Batch(kws) as b:
            b.set_chunk_bytes(size)
            for i, s in enumerate(sig):
                b.instance(i).set_sigma(s)
            b.iterate(2, 0.0)
            got.append([(b.instance(i).get_gloc(), b.instance(i).get_sigma())
                        for i in range(len(sizes))])
    for one, many in zip(*got):
        for p, q in zip(one, many):
            assert np.max(np.abs(p - q)) < 1e-10 * np.max(np.abs(p))
