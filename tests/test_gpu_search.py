"""The neighbour search at the edges of its tiles, chunks and paths: the lists
equal the oracle's sets exactly, whatever path a tile takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.load()
    torch.cuda.set_device(0)


def _h(n, k):
    """h of a unit cube of n particles with about k neighbours inside 2 h."""
    return 0.5 * (k / (4.18879 * n)) ** (1.0 / 3.0)


def _cloud(n, k, spread=0.0, periodic=(0, 0, 0), seed=0):
    h = _h(n, k)
    return I.random_cloud(n, seed=seed, h_min=h * (1 - spread), h_max=h * (1 + spread),
                          periodic=periodic)


def _short_box(nc, periodic, spread=0.0, n=900):
    """A unit box of nc cells per axis (nc = 2 is the shortest allowed)."""
    h = 0.499 / nc
    return I.random_cloud(n, seed=nc, h_min=h * (1 - spread), h_max=h, periodic=periodic)


def _far(where):
    """Some particles of an open box far outside it, one at a coordinate whose
    square FP32 does not hold."""
    ic = _cloud(3000, 60, 0.3, seed=5)
    ic.x[:20] += where
    ic.y[20:40] -= where
    ic.z[40] = 1e25
    return ic


def _lattice(jitter):
    """Lattice whose outer shell lies exactly on the reach (settled in FP64)."""
    return I.lattice_periodic(16, spacing=2.0 ** -4, jitter=jitter)


CASES = {
    # sizes around a tile, with sixteen waves on each tile
    **{f"n_{n}": (lambda n=n: _cloud(n, min(40, n)), 512) for n in (1, 63, 64, 65, 129)},
    # either side of the line between sixteen waves and four per tile
    "cu_tiles": (lambda: _cloud(16384, 60, 0.3), 256),
    "more_tiles": (lambda: _cloud(16385, 60, 0.3), 256),
    # four waves: unions of several chunks, images, few rows
    "shared_several_chunks": (lambda: _cloud(20000, 700, 0.2), 2048),
    "shared_chunks_uniform": (lambda: _cloud(20000, 900, 0.0, (0, 1, 0)), 2048),
    "shared_box": (lambda: _short_box(5, (1, 1, 1), 0.3, 17000), 1024),
    "shared_short_lists": (lambda: _cloud(17000, 80, 0.2), 24),
    # either side of the line between four waves and one wave per tile
    "shared_tiles": (lambda: _cloud(131072, 40, 0.3), 256),
    "single_tiles": (lambda: _cloud(131073, 40, 0.3), 256),
    "single_tiles_uniform": (lambda: _cloud(140001, 60, 0.0, (0, 0, 1)), 256),
    "single_tiles_periodic": (lambda: _cloud(150000, 30, 0.2, (1, 1, 1)), 256),
    # unions of more candidates than LDS has bits for, one wave and four
    "several_chunks": (lambda: _cloud(6000, 700, 0.2), 2048),
    "several_chunks_uniform": (lambda: _cloud(5000, 900, 0.0, (0, 1, 0)), 2048),
    "single_several_chunks": (lambda: _cloud(140000, 150, 0.2), 512),
    # fewer rows than neighbours
    "short_lists": (lambda: _cloud(4000, 80, 0.2), 24),
    # periodic axes of two to five cells: both images of a candidate in play
    **{f"box_{nc}_{p[0]}{p[1]}{p[2]}": (lambda nc=nc, p=p: _short_box(nc, p, 0.3), 1024)
       for nc in (2, 3, 4, 5) for p in ((1, 1, 1), (0, 0, 1))},
    "box_3_uniform": (lambda: _short_box(3, (1, 1, 0), n=3001), 2048),
    # many nearly empty cells: more distinct cells than the union build takes
    "sparse": (lambda: _cloud(20000, 0.05, 0.5), 64),
    "single_sparse": (lambda: _cloud(140000, 0.3, 0.5, (0, 1, 0)), 64),
    "far_outside": (lambda: _far(50.0), 512),
    "far_outside_1e9": (lambda: _far(1e9), 512),
    # every shell pair decided in FP64
    "on_the_shell": (lambda: _lattice(0.0), 128),
    "near_the_shell": (lambda: _lattice(1e-7), 128),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lists_are_the_oracles(name):
    make, max_nb = CASES[name]
    ic = make()
    print(f"search {name} n={ic.n}", flush=True)
    off, ids = O.neighbors(ic.x, ic.y, ic.z, ic.h, ic.lo, ic.hi, ic.periodic)
    ctx = S.Context(ic.n, max_nb)
    st = S.SphState(ic, max_nb)
    S.sph_build_cells(ctx, st)
    S.sph_find_neighbors(ctx, st)
    n_ref = np.diff(off)
    if n_ref.max(initial=0) > max_nb:
        with pytest.raises(S.SphError):
            S.sph_ctx_check(ctx)
    else:
        S.sph_ctx_check(ctx)
    count = st.host(["count"])["count"]
    assert np.array_equal(count, n_ref)
    # the lists ascend in the library's order, and hold only what fits
    idx = st.t["idx"].view(max_nb, ic.n).cpu().numpy()
    got_id = st.t["id"].cpu().numpy()
    cnt = np.minimum(count[got_id], max_nb)
    rows = np.arange(max_nb)[:, None] < cnt[None, :]
    assert (np.diff(idx, axis=0)[rows[1:]] > 0).all()
    if n_ref.max(initial=0) <= max_nb:
        goff, gids = S.sph_export_neighbors(ctx, st)
        assert np.array_equal(goff, off) and np.array_equal(gids, ids)
    else:
        for k in range(0, ic.n, 7):  # the first max_nb of each set, in the library's order
            i = int(np.nonzero(got_id == k)[0][0])
            where = np.empty(ic.n, dtype=np.int64)
            where[got_id] = np.arange(ic.n)
            want = np.sort(where[ids[off[k]:off[k + 1]]])[:max_nb]
            assert np.array_equal(idx[: cnt[i], i], want)
