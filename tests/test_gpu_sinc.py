"""The sinc kernels' shape at the edges of its series."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

pytestmark = pytest.mark.gpu

Q = [1e-12, 1e-3, 0.5, 1 - 1e-15, 1.0, 1 + 1e-15, 1.2, 1.5, 1.9, 1.999, 2 - 1e-9, 2.5]


@pytest.mark.parametrize("exponent", [3, 4, 5, 8, 12])
def test_shape_of_pairs(exponent):
    """Pairs of particles q h apart, each far from the others: the density over
    that of a lone particle is 1 + S(q)^n. S is good to 4e-16, the n factors and
    the sum round n + 2 times: within 2 n times 2.2e-16 of it, and one more for
    the position that carries q (dS/dq is below 0.7)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    print(f"sinc exponent={exponent}", flush=True)
    h, n = 2.0 ** -8, 2 * len(Q) + 1
    ic = I.random_cloud(n, seed=0, h_min=h, h_max=h)
    at = np.arange(len(Q)) * 0.0625 + 0.03125
    ic.x[:] = np.concatenate([at, at, [0.875]])
    ic.y[:] = 0.0
    ic.y[len(Q):-1] = np.array(Q) * h  # (exact differences)
    ic.z[:] = 0.5
    ic.m[:] = 1.0
    prm = S.make_params(dataclasses.replace(ic.params, kernel=S.SPH_KERNEL_SINC,
                                            sinc_n=exponent))
    ctx = S.Context(4096, 16)
    st = S.SphState(ic, 16)
    S.sph_build_cells(ctx, st)
    S.sph_find_neighbors(ctx, st)
    S.sph_density(ctx, st, prm)
    S.sph_ctx_check(ctx)
    rho = st.host(["rho"])["rho"]
    ratio = rho[:-1] / rho[-1]
    x = np.array(Q, dtype=np.longdouble) * (np.longdouble(np.pi) / 2)
    want = np.where(np.array(Q) < 2, 1 + (np.sin(x) / x) ** exponent, 1).astype(np.float64)
    tol = (2 * exponent + 4) * 2.2e-16
    assert np.max(np.abs(ratio[: len(Q)] - want)) <= tol
    assert np.max(np.abs(ratio[len(Q):] - want)) <= tol
