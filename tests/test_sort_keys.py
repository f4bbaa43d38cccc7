"""The serving engine's sort keys: the last radix pass ranks particles by the
sorted bits alone and counts them by the whole digit, so no key may have a bit
above the sorted ones, the key of a run being dropped included."""
import os
import subprocess

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1809_08013_amd import build as B  # noqa: E402
from paper_1809_08013_amd import inputs as I  # noqa: E402
from paper_1809_08013_amd import sph as S  # noqa: E402

SRC = r"""
#include <cstdio>
#include "sph_internal.h"
using namespace sph;
int main()
{
    // the largest key of a slot: its last cell's last slice
    auto last = [](uint32_t slot) { return (slot << kEnsSlotShift) | ((1u << kEnsSlotShift) - 1u); };
    printf("%d %llu %llu %d\n", kEnsKeyBits, (unsigned long long)kEnsDropKey,
           (unsigned long long)last(kEnsMaxSlots - 1), kRadixBits);
    for (uint32_t s = 0; s < (uint32_t)kEnsMaxSlots; ++s) printf("%u ", last(s));
    return 0;
}
"""


def test_no_key_has_bits_above_the_sorted_ones(tmp_path):
    """Compiled from the library's own header; then the last pass over one wave of
    keys of each slot and dropped ones, counted by the digit and ranked by the
    sorted bits, has to place every key once."""
    src, exe = tmp_path / "keys.hip", tmp_path / "keys"
    src.write_text(SRC)
    subprocess.check_call([B.HIPCC, "--offload-host-only", "-std=c++17", f"-I{B.INCLUDE}",
                           f"-I{B.CSRC}", str(src), "-o", str(exe)])
    v = [int(w) for w in subprocess.check_output([str(exe)]).split()]
    bits, drop, largest, radix = v[:4]
    last = np.array(v[4:], dtype=np.int64)
    assert drop >> bits == 0 and largest >> bits == 0
    assert drop > largest  # dropped particles sort behind every live one
    shift = (bits - 1) // radix * radix
    low = (1 << (bits - shift)) - 1
    for slot in range(last.size):
        keys = np.concatenate([np.full(20, last[slot]), np.full(44, drop)])
        digit = (keys >> shift) & ((1 << radix) - 1)
        base = np.concatenate([[0], np.cumsum(np.bincount(digit, minlength=1 << radix))])
        rank = np.array([np.sum((digit[:i] & low) == (digit[i] & low)) for i in range(64)])
        assert np.array_equal(np.sort(base[digit] + rank), np.arange(64)), slot


@pytest.mark.gpu
def test_every_slot_taken():
    """More runs than the 511 slots, ending at different steps, so that runs of the
    last slots stay while others are dropped: each is bitwise the run alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    kinds = [I.square_patch(side, nz=nz, kmax=9) for side, nz in ((4, 7), (3, 8), (5, 7), (4, 9))]
    steps = (400, 430, 470, 520, 600)  # (the first ones end after the last is submitted)
    alone = {}
    for k, ic in enumerate(kinds):
        prm = S.make_params(ic.params)
        ctx, st = S.Context(ic.n, 128), S.SphState(ic, 128)
        S.sph_init_forces(ctx, st, prm, set_rho_ref=True)
        for q in range(1, max(steps) + 1):
            S.sph_step(ctx, st, prm)
            if q in steps:
                alone[k, q] = {**st.host(["x", "vx", "u", "rho"]), "diag": st.diag.copy()}
        S.sph_ctx_check(ctx)
    ens = S.Ensemble(256 << 20, max_slots=511, max_n_per_run=175)
    try:
        runs = [(i % 4, steps[i % 5]) for i in range(600)]
        tickets = [ens.submit(kinds[k], q) for k, q in runs]
        for i, ((k, q), t) in enumerate(zip(runs, tickets)):
            got = ens.wait(t, kinds[k].n)
            assert got["status"] == S.SPH_OK and got["steps_done"] == q
            for name, want in alone[k, q].items():
                assert np.array_equal(got[name], want), (i, k, q, name)
        print("most runs in one step:", ens.stats()["peak_runs"], flush=True)
        assert ens.stats()["peak_runs"] > 504
    finally:
        ens.close()
