"""The patch's pressure series over several row chunks, which threads evaluate, equals
the same rows taken one chunk at a time."""
import threading
from concurrent.futures import ThreadPoolExecutor

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


def _most_threads_in_a_product(monkeypatch, work):
    """Largest number of threads inside a matrix product together while work runs."""
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
    work()
    return most[0]


def test_products_one_at_a_time(monkeypatch):
    """(The values above go wrong only now and then when they are not.)"""
    rng = np.random.default_rng(1)
    x, y = rng.random((2, 6 * CHUNK)) - 0.5
    assert _most_threads_in_a_product(
        monkeypatch, lambda: I.square_patch_pressure(x, y, kmax=19)) == 1


def test_products_of_callers_threads(monkeypatch):
    """Several threads that make an input each, as a client of the serving engine may."""
    rng = np.random.default_rng(2)
    x, y = rng.random((2, 300_000)) - 0.5

    def work():
        with ThreadPoolExecutor(max_workers=6) as ex:
            list(ex.map(lambda _: I.square_patch_pressure(x, y, kmax=49), range(18)))

    assert _most_threads_in_a_product(monkeypatch, work) == 1
