"""Small runs share a particle among several lanes: the sums are bit for bit
those of one lane per particle, which a run of more particles takes."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

pytestmark = pytest.mark.gpu

ONE_LANE = 114_689   # particles of the smallest run at one lane per particle
DENSITY = 4e5        # particles per unit volume: about 50 inside 2 h
OUT = ("rho", "ax", "ay", "az", "dudt", "mumax")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.load()
    torch.cuda.set_device(0)


def _cloud(n, total, spread):
    """n particles of a unit box at x < 0.4, and others far from them up to
    `total`: the first n have the same cells and lists whatever the total."""
    rng = np.random.default_rng(n)
    h0 = 0.5 * (50 / (4.18879 * DENSITY)) ** (1 / 3)
    ic = I.random_cloud(total, seed=n, h_min=h0, h_max=h0)
    a = min(0.4, (n / DENSITY) ** (1 / 3))
    b = min(0.999, (n / (DENSITY * a)) ** 0.5)
    pos = rng.random((n, 3)) * [a, b, b]
    more = np.random.default_rng(n + 1).random((total - n, 3)) * [0.3, 1, 1] + [0.7, 0, 0]
    for k, axis in enumerate("xyz"):
        getattr(ic, axis)[:] = np.concatenate([pos[:, k], more[:, k]])
        getattr(ic, "v" + axis)[:n] = rng.standard_normal(n)
    ic.h[1:n] *= 1 - spread * rng.random(n - 1)
    ic.m[:] = 1 / DENSITY
    ic.m[:n] *= 1 + 0.1 * rng.random(n)
    ic.u[:n] = 1 + rng.random(n)
    return ic


def _forces(ic, n, prm):
    ctx = S.Context(ONE_LANE, 160)  # (the grid of both runs)
    st = S.SphState(ic, 160)
    S.sph_build_cells(ctx, st)
    S.sph_find_neighbors(ctx, st)
    S.sph_density(ctx, st, prm)
    S.sph_eos(ctx, st, prm)
    S.sph_momentum_energy(ctx, st, prm)
    S.sph_ctx_check(ctx)
    return {k: v[:n] for k, v in st.host(list(OUT) + ["count"]).items()}


CASES = [(n, p, k, s) for n in (1, 5, 65, 3001) for p in (0, 1) for k in (0, 1, 2)
         for s in (0.0, 0.3)]
CASES += [(n, p, 0, s) for n in (12_288, 12_289, 114_688) for p in (0, 1) for s in (0.0, 0.3)]


@pytest.mark.parametrize("n,precision,kernel,spread", CASES)
def test_shared_particle_sums(n, precision, kernel, spread):
    prm = S.make_params(dataclasses.replace(I.random_cloud(8).params, kernel=kernel, sinc_n=5),
                        precision)
    print(f"split n={n} precision={precision} kernel={kernel} spread={spread}", flush=True)
    got = _forces(_cloud(n, n, spread), n, prm)
    want = _forces(_cloud(n, ONE_LANE, spread), n, prm)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    if n > 1000:
        assert got["count"].mean() > 20 and np.abs(got["ax"]).max() > 0


def _stepping(n, total):
    """_cloud with a few hot particles (deep bins) and the others of the total
    alone on a lattice, at rest, with a step in the middle of the range."""
    ic = _cloud(n, n, 0.0)
    ic.u[: max(1, n // 100)] *= 9.0
    for axis in "xyz":
        getattr(ic, "v" + axis)[:] *= 0.1
    if total == n:
        return ic
    more = total - n
    side = int(np.ceil((more / 0.25) ** (1 / 3)))
    k = np.arange(more)
    big = I.random_cloud(total, seed=0, h_min=ic.h[0], h_max=ic.h[0])
    for name, a in ic.arrays().items():
        if name != "id":
            getattr(big, name)[:n] = a
    big.x[n:] = 0.7 + (k // side ** 2 + 0.5) / side
    big.y[n:] = (k // side % side + 0.5) / side
    big.z[n:] = (k % side + 0.5) / side
    big.h[n:] = 0.3 * ic.h[0]
    big.u[n:] = 0.09 * 1.5
    for axis in "xyz":
        getattr(big, "v" + axis)[n:] = 0.0
    return big


@pytest.mark.parametrize("n", [300, 3001])
def test_block_steps_by_what_closes(n):
    """Individual time steps choose their launches by how many particles close:
    bit for bit the same particles with few others and with many, which close
    only with the shallow bins."""
    print(f"block steps n={n}", flush=True)
    out = []
    for total in (n, ONE_LANE):
        ic = _stepping(n, total)
        assert ic.x.max() < 1.0
        prm = S.make_params(ic.params)
        ctx = S.Context(ONE_LANE, 160)
        st = S.SphState(ic, 160)
        S.sph_init_forces(ctx, st, prm)
        subs = [S.sph_step_blocks(ctx, st, prm, 4) for _ in range(2)]
        S.sph_ctx_check(ctx)
        got = {k: v[:n] for k, v in st.host(["x", "vx", "u", "rho", "ax", "dudt", "bin"]).items()}
        if total > n:  # alone, and in a shallower bin than the hot ones
            full = st.host(["count", "bin"])
            assert full["count"][n:].max() == 0
            assert full["bin"][n:].max() < full["bin"][:n].max()
        out.append((subs, got))
    assert out[0][0] == out[1][0] and max(out[0][0]) > 1
    for k in out[0][1]:
        assert np.array_equal(out[0][1][k], out[1][1][k]), k
