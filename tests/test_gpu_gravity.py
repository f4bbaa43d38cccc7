"""The direct sum where it is cut into shares and where it is not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.0, 0.01])
@pytest.mark.parametrize("n", [1, 3, 255, 257, 4097, 131073, 262145])
def test_direct_sum_shares(n, eps):
    """Every particle (a sample of the large ones) within 1e-13 of the sum of
    the terms' magnitudes: each term is good to a few ulp and the sum's order
    differs, so the error is that of a pairwise or running sum, at most
    sqrt(n) u = 6e-14 of that scale."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    print(f"direct sum n={n} eps={eps}", flush=True)
    ic = I.evrard(n, seed=3)
    if n > 1000:  # coincident particles contribute nothing to each other
        ic.x[7], ic.y[7], ic.z[7] = ic.x[5], ic.y[5], ic.z[5]
    ctx = S.Context(n, 16)
    st = S.SphState(ic, 16)
    S.sph_gravity_direct(ctx, st, eps)
    S.sph_ctx_check(ctx)
    got = st.host(["gx", "gy", "gz"])
    sel = np.arange(n) if n < 5000 else np.random.default_rng(0).choice(n, 300, replace=False)
    gx, gy, gz, scale = O.gravity_direct_subset(ic.x, ic.y, ic.z, ic.m, sel, eps)
    if eps == 0.0:  # 0/0 in the oracle's definition for the two: finite here
        undefined = np.isnan(scale)
        assert undefined.sum() <= 2
        assert all(np.isfinite(got[a][sel]).all() for a in ("gx", "gy", "gz"))
        sel, gx, gy, gz, scale = (v[~undefined] for v in (sel, gx, gy, gz, scale))
    scale = np.where(scale > 0, scale, 1.0)
    for a, b in (("gx", gx), ("gy", gy), ("gz", gz)):
        assert np.max(np.abs(got[a][sel] - b) / scale) <= 1e-13


@pytest.mark.parametrize("leaf", [8, 16, 64])
@pytest.mark.parametrize("n", [1, 2, 32, 33, 64, 65, 130, 9001])
def test_tree_groups_and_leaves(n, leaf):
    """The octree at the edges of its groups (32, 64 particles), with the smallest, the
    usual and the largest leaves: within 1e-12 of the terms'
    magnitudes, the accuracy of the node terms' eight FP64 factors over a few
    hundred terms."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    print(f"tree n={n} leaf={leaf}", flush=True)
    ic = I.evrard(n, seed=4)
    gx, gy, gz, scale, _ = O.gravity_tree(ic.x, ic.y, ic.z, ic.m, 0.01, 0.6, leaf)
    ctx = S.Context(n, 16)
    st = S.SphState(ic, 16)
    S.sph_gravity_tree(ctx, st, 0.01, 0.6, leaf)
    S.sph_ctx_check(ctx)
    got = st.host(["gx", "gy", "gz"])
    scale = np.where(scale > 0, scale, 1.0)
    for a, b in (("gx", gx), ("gy", gy), ("gz", gz)):
        assert np.max(np.abs(got[a] - b) / scale) <= 1e-12


@pytest.mark.parametrize("eps", [0.0, 0.01])
@pytest.mark.parametrize("n", [2, 79, 80, 81, 82])
def test_direct_sum_of_few(n, eps):
    """Either side of the particles from which on the sum is cut into shares, within
    the bound of test_direct_sum_shares."""
    test_direct_sum_shares(n, eps)
