"""The patch's pressure series over several row chunks, which threads evaluate, equals
the same rows taken one chunk at a time."""
import threading

import numpy as np

from paper_1809_08013_amd import inputs as I

CHUNK = 1 << 20


def test_chunks_in_threads_equal_single_chunks():
    rng = np.random.default_rng(0)
    x, y = rng.random((2, 4 * CHUNK + 77)) - 0.5
    want = np.concatenate([I.square_patch_pressure(x[a:a + CHUNK], y[a:a + CHUNK], kmax=19)
                           for a in range(0, x.size, CHUNK)])
    for _ in range(3):
        assert np.array_equal(I.square_patch_pressure(x, y, kmax=19), want)


def test_products_one_at_a_time(monkeypatch):
    """No two threads are inside a matrix product together (the values above go wrong
    only now and then when they are)."""
    inside, most, lock = [0], [0], threading.Lock()

    class Coef(np.ndarray):
        def __array_ufunc__(self, ufunc, method, *args, **kw):
            args = [np.asarray(a) for a in args]
            if ufunc is np.matmul:
                with lock:
                    inside[0] += 1
                    most[0] = max(most[0], inside[0])
                try:
                    return getattr(ufunc, method)(*args, **kw)
                finally:
                    with lock:
                        inside[0] -= 1
            return getattr(ufunc, method)(*args, **kw).view(Coef)

    grid = np.meshgrid

    def meshgrid(*a, **kw):
        return [m.view(Coef) for m in grid(*a, **kw)]

    monkeypatch.setattr(np, "meshgrid", meshgrid)
    rng = np.random.default_rng(1)
    x, y = rng.random((2, 6 * CHUNK)) - 0.5
    I.square_patch_pressure(x, y, kmax=19)
    assert most[0] == 1
