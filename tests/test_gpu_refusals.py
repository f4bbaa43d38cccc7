"""A step whose argument is refused part of the way leaves what its separate calls
leave: everything before the refused one has been done."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [S.SPH_FP64, S.SPH_FP32_PAIR])
@pytest.mark.parametrize("first", [True, False])
def test_refused_momentum_leaves_the_eos(first, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    ic = I.square_patch(12)
    prm = S.make_params(ic.params, precision)
    out = []
    for parts in (False, True):
        ctx, st = S.Context(ic.n, 128), S.SphState(ic, 128)
        if not first:
            S.sph_init_forces(ctx, st, prm)
        for k in ("p", "c", "pr2"):
            st.t[k].fill_(-1.0)
        accel = S.Accel(*[C.c_void_p(st.t[k].data_ptr()) for k in ("ax", "ay", "az", "dudt")], None)
        call = (lambda fn, *a: fn(ctx.h, C.byref(st.particles), C.byref(st.box), *a))
        if parts:
            if not first:
                S.sph_integrate(ctx, st, S.SPH_KICK_DRIFT)
            S.sph_build_cells(ctx, st)
            S.sph_find_neighbors(ctx, st)
            S.sph_density(ctx, st, prm)
            if first:
                st.t["rho_ref"].copy_(st.t["rho"][: ic.n])
            S.sph_eos(ctx, st, prm)
            s = call(ctx.lib.sph_momentum_energy, C.byref(st.nbrs), C.byref(prm),
                     C.byref(st.fields), C.byref(accel))
        else:
            rest = (C.byref(st.nbrs), C.byref(prm), C.byref(st.fields), C.byref(accel))
            dt, diag = (C.c_void_p(st.t[k].data_ptr()) for k in ("dt", "diag"))
            if first:
                s = call(ctx.lib.sph_init_forces, st.h_max, *rest, 1, dt, diag)
            else:
                s = call(ctx.lib.sph_step, st.h_max, *rest, dt, diag)
        assert s == S.SPH_E_INVALID
        assert b"mumax" in ctx.lib.sph_last_error(ctx.h)
        S.sph_ctx_check(ctx)
        out.append(st.host())
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
    assert (out[0]["c"] > 0).all()
