"""The sinc shape and its slope as the kernels compute them (the library's own header
compiled for the host), against 64 bits of mantissa."""
import subprocess

import numpy as np

from paper_1809_08013_amd import build as B

SRC = r"""
#include <cstdio>
#include <vector>
#include "sinc.h"
int main()
{
    double q;
    std::vector<double> out;
    auto est = [](double b) { return (double)(1.0f / (float)b); };
    while (fread(&q, sizeof q, 1, stdin) == 1) {
        const double s = sph::sinc_s(q, est);
        out.push_back(s);
        out.push_back(sph::sinc_ds(q));
    }
    fwrite(out.data(), sizeof(double), out.size(), stdout);
    return 0;
}
"""


def _reference(q):
    """S and dS/dq in extended precision: the series in x^2 where their terms do not
    cancel, beyond by the sine and cosine of pi (2 - q) / 2."""
    half_pi = np.longdouble("1.57079632679489661923132169163975144")
    q = q.astype(np.longdouble)
    x2 = (half_pi * q) ** 2
    s, d, t = np.zeros_like(q), np.zeros_like(q), np.ones_like(q)
    for k in range(26):
        s += t
        d += (2 * k) * t
        t = -t * x2 / ((2 * k + 2) * (2 * k + 3))
    y = half_pi * (2 - q)
    sin, cos = np.zeros_like(q), np.zeros_like(q)
    t = np.ones_like(q)
    for k in range(24):
        cos += t
        sin += t * y / (2 * k + 1)
        t = -t * y * y / ((2 * k + 1) * (2 * k + 2))
    far = q > 1
    s = np.where(far, sin / (half_pi * q), s)
    d = np.where(q > 1.3, -(cos + s) / q, d / np.where(q > 0, q, 1))
    return s, d


def test_shape_and_slope(tmp_path):
    """u = 2^-53. S: the series 1.5 u on [0, 1]; beyond, half an ulp each for the
    quotient, its correction and the product more: 2.7 u. dS/dq: coefficients and
    partial sums round to 1.3 u of a result that is 0.4 of their sum, the argument adds
    0.6 u, the last sum and the factor half an ulp each: 3 u."""
    src, exe = tmp_path / "s.hip", tmp_path / "s"
    src.write_text(SRC)
    subprocess.check_call([B.HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-mfma",
                           "-ffp-contract=off", f"-I{B.INCLUDE}", f"-I{B.CSRC}", str(src), "-o",
                           str(exe)])
    q = np.concatenate([(np.arange(400_000) + 0.37) / 200_000, 10.0 ** -np.arange(1.0, 13.0),
                        2 - 2.0 ** -np.arange(2.0, 50.0),
                        *[np.nextafter(e, [0.0, 4.0]) for e in (0.5, 1.0, 1.5)], [0.5, 1.0, 1.5]])
    got = np.frombuffer(subprocess.run([str(exe)], input=q.tobytes(), capture_output=True,
                                       check=True).stdout).reshape(-1, 2)
    s, d = _reference(q)
    u = 2.0 ** -53
    es, ed = np.abs(got[:, 0] / s - 1), np.abs(got[:, 1] / d - 1)
    print("largest relative errors", float(es.max()), float(ed.max()))
    assert es.max() <= 2.7 * u
    assert ed.max() <= 3.0 * u
