"""The neighbour search where a tile's union of cells is about as large as the
search holds: the lists equal the oracle's sets, whatever path a tile takes."""
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


def _cloud(n, k, spread=0.0, periodic=(0, 0, 0), seed=1):
    h = 0.5 * (k / (4.18879 * n)) ** (1.0 / 3.0)
    return I.random_cloud(n, seed=seed, h_min=h * (1 - spread), h_max=h * (1 + spread),
                          periodic=periodic)


def _check(ic, max_nb):
    off, ids = O.neighbors(ic.x, ic.y, ic.z, ic.h, ic.lo, ic.hi, ic.periodic)
    ctx = S.Context(ic.n, max_nb)
    st = S.SphState(ic, max_nb)
    S.sph_build_cells(ctx, st)
    S.sph_find_neighbors(ctx, st)
    S.sph_ctx_check(ctx)
    goff, gids = S.sph_export_neighbors(ctx, st)
    assert np.array_equal(goff, off) and np.array_equal(gids, ids)


def _union_sizes(ic):
    """Non-empty cells within one cell of a tile's cells, for every tile: the
    largest union the search may see (it drops cells out of reach)."""
    nc = np.array([int((b - a) / (2.0 * ic.h.max() * (1 + 1e-9))) for a, b in zip(ic.lo, ic.hi)])
    c = np.stack([np.clip(((p - a) * (m / (b - a))).astype(int), 0, m - 1)
                  for p, a, b, m in zip((ic.x, ic.y, ic.z), ic.lo, ic.hi, nc)], axis=1)

    def spread(v):
        return sum(((v >> b) & 1) << (3 * b) for b in range(10))

    morton = spread(c[:, 0]) | spread(c[:, 1]) << 1 | spread(c[:, 2]) << 2
    c = c[np.argsort(morton, kind="stable")]
    full = np.zeros(tuple(nc), dtype=bool)
    full[tuple(c.T)] = True
    off = np.stack(np.meshgrid(*[[-1, 0, 1]] * 3, indexing="ij"), -1).reshape(-1, 3)
    sizes = []
    for t in range(0, ic.n, 64):
        near = (np.unique(c[t:t + 64], axis=0)[:, None, :] + off).reshape(-1, 3)
        for a in range(3):
            if ic.periodic[a]:
                near[:, a] %= nc[a]
        near = np.unique(near[((near >= 0) & (near < nc)).all(axis=1)], axis=0)
        sizes.append(int(full[tuple(near.T)].sum()))
    return np.array(sizes)


@pytest.mark.parametrize("spread,k,periodic", [(0.0, 52, (0, 0, 1)), (0.0, 52, (1, 1, 1)),
                                               (0.3, 25, (0, 0, 0)), (0.0, 25, (0, 0, 0))])
def test_unions_about_as_large_as_held(spread, k, periodic):
    """One wave per tile holds 104 cells: tiles with fewer, with just that many, and
    (in the last case) with more."""
    ic = _cloud(150_000, k, spread, periodic)
    n = _union_sizes(ic)
    print(f"unions k={k} spread={spread} up to 92: {(n <= 92).sum()}, 104: {(n <= 104).sum()}, "
          f"more: {(n > 104).sum()}", flush=True)
    assert (n <= 92).any() and ((n > 92) & (n <= 104)).any()
    _check(ic, int(2.5 * k * (1 + spread) ** 3) + 24)


@pytest.mark.parametrize("n", [65_536, 65_537, 131_072])
@pytest.mark.parametrize("k,spread", [(2, 0.0), (17, 0.0), (22, 0.0), (6, 0.3), (10, 0.3)])
def test_thin_cells(n, k, spread):
    """Either side of 4.5 particles per cell and of the tiles from which on a run
    with fewer takes one wave per tile."""
    print(f"thin n={n} k={k} spread={spread}", flush=True)
    _check(_cloud(n, k, spread, (0, 0, 1)), int(3 * k * (1 + spread) ** 3) + 24)


@pytest.mark.parametrize("n", [5_000, 20_000, 140_000])
@pytest.mark.parametrize("spread,periodic", [(0.0, (0, 0, 0)), (0.3, (0, 0, 0)), (0.3, (1, 0, 1))])
def test_positions_that_are_not_numbers(n, spread, periodic):
    """NaN, infinite and huge coordinates, first in their tile and in the middle of one,
    with sixteen, four and one wave per tile: such particles have no neighbours but
    those of the same huge coordinate, the others have the lists they have without
    them."""
    print(f"not numbers n={n} spread={spread} {periodic}", flush=True)
    ic = _cloud(n, 60, spread, periodic)
    bad = np.random.default_rng(2).choice(n, 24, replace=False)
    values = [np.nan, np.inf, -np.inf, 1e300]
    for q, i in enumerate(bad):
        (ic.x, ic.y, ic.z)[q % 3][i] = values[q % 4]
        if q % 5 == 0:
            ic.x[i] = ic.y[i] = ic.z[i] = np.nan
    good = np.setdiff1d(np.arange(n), bad)
    off, ids = O.neighbors(ic.x[good], ic.y[good], ic.z[good], ic.h[good], ic.lo, ic.hi, ic.periodic)
    want = [np.empty(0, dtype=np.int64)] * n
    for k, i in enumerate(good):
        want[i] = good[ids[off[k]:off[k + 1]]]
    with np.errstate(invalid="ignore", over="ignore"):
        for i in bad:
            r2 = sum((p[i] - p[bad]) ** 2 for p in (ic.x, ic.y, ic.z))
            near = r2 < (2.0 * np.maximum(ic.h[i], ic.h[bad])) ** 2
            want[i] = np.sort(bad[near & (bad != i)])
    max_nb = int(2.5 * 60 * (1 + spread) ** 3)
    ctx, st = S.Context(n, max_nb), S.SphState(ic, max_nb)
    S.sph_build_cells(ctx, st)
    S.sph_find_neighbors(ctx, st)
    S.sph_ctx_check(ctx)
    goff, gids = S.sph_export_neighbors(ctx, st)
    assert np.array_equal(np.diff(goff), [w.size for w in want])
    assert np.array_equal(gids, np.concatenate(want))


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("n", [5_000, 140_000])
def test_lengths_that_are_not_numbers(n, value):
    """An h that is no number is above the promised bound: the calls end and the check
    says so; a context that has seen it works on."""
    ic = _cloud(n, 40, 0.3)
    h_max = float(ic.h.max())
    ic.h[::97] = value
    ctx, st = S.Context(n, 256), S.SphState(ic, 256)
    S.sph_build_cells(ctx, st, h_max)
    S.sph_find_neighbors(ctx, st)
    with pytest.raises(S.SphError) as e:
        S.sph_ctx_check(ctx)
    assert e.value.status == S.SPH_E_DOMAIN
    _check(_cloud(n, 40, 0.3), 256)
