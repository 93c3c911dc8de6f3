"""The FP64 form's near-field table (host code, no GPU): three points of every
interval, evaluated as the kernel does, against the sum of all Gaussians of the
split in extended precision, for both bases (b = 2^(1/2) and 2^(1/4)) and short,
usual and long cutoffs.

Bar: the coefficients are rounded to 53 bits from an interpolation whose
truncation is below 1e-16 of the bare Coulomb kernel, Horner in FP64 adds about
two roundings, and the weights and widths it is built from carry one each under
sums of both signs no larger than the kernel: within 4e-15 of it."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2512_24970_amd import rbsog as R

LD = np.longdouble


@pytest.mark.parametrize("eps", [1e-5, 1e-7])
@pytest.mark.parametrize("r_shell", [2.5, 8.0, 10.0, 11.0, 47.0])
def test_near_table64_matches_the_split(eps, r_shell):
    tab = R.rbsog_near_table64(eps, r_shell)
    sp = R.rbsog_sog_params(eps, r_shell)
    assert sp["b"] == pytest.approx(2 ** 0.5 if eps == 1e-5 else 2 ** 0.25, rel=1e-15)
    coef, e0 = tab["coef"], tab["e0"]
    nbin = len(coef) // 32
    assert len(coef) == 32 * nbin and 2.0 ** (e0 + nbin) > r_shell ** 2
    sg = LD(sp["s"]) * LD(sp["b"]) ** np.arange(sp["M"] + 1)
    w = sp["w"].astype(LD)
    worst = 0.0
    for q in range(len(coef)):
        lo, h = np.ldexp(1.0 + (q % 32) / 32, e0 + q // 32), np.ldexp(1.0 / 64, e0 + q // 32)
        for x in (-1.0, 0.37, 1.0 - 2.0 ** -40):
            s = (lo + h) + x * h
            t = s - (lo + h)
            g = np.exp(-LD(s) / (2 * sg * sg))
            for k, ref, bare in ((0, LD(s) ** LD(-1.5) - (w / (sg * sg) * g).sum(), s ** -1.5),
                                 (8, LD(s) ** LD(-0.5) - (w * g).sum(), s ** -0.5)):
                v = 0.0
                for c in coef[q, k:k + 8][::-1]:
                    v = v * t + c
                worst = max(worst, abs(float(LD(v) - ref)) / bare)
    print(f"eps {eps} r_shell {r_shell}: {worst:.2e} of the bare kernel")
    assert worst < 4e-15
