"""The pair histogram and the displacement sums at the edges of their work
split: ion counts around a wavefront's 16 atoms and a workgroup's 256, one bin,
bins narrower than an FP32 ulp of the radius allows to guess, a sub-shell
r_max, and repeated calls of growing and shrinking size on one context.
Counts are integers and must match the oracle's scan over all pairs exactly;
the MSD is a sum of N squares (1e-13)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [510, 514, 526, 770, 1024])
@pytest.mark.parametrize("precision", [R.FP64, R.MIXED])
def test_counts_and_msd(n, precision):
    import torch
    print(f"case: observe edges n {n} precision {precision}", flush=True)
    cfg = W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3))
    dev = torch.device("cuda", 0)
    ctx = R.Context(0)
    ctx.rbsog_set_system(R.make_params(cfg["sys"], precision, n_atoms=n),
                         *(torch.as_tensor(cfg[k], device=dev) for k in ("types", "pos", "vel")))
    osys = O.System(cfg["sys"], cfg["types"], cfg["pos"], cfg["vel"])
    for r_max, bins in ((10.0, 4096), (10.0, 1), (4.99, 37), (10.0, 250)):
        got = ctx.rbsog_rdf_counts(r_max, bins)
        assert np.array_equal(got, osys.rdf_counts(r_max, bins)), (r_max, bins)
        assert np.array_equal(got, ctx.rbsog_rdf_counts_noalloc(r_max, bins))
    ctx.rbsog_msd(mark=True)
    move = np.random.default_rng(n).uniform(-0.2, 0.2, (n, 3))
    ctx.rbsog_set_positions(torch.as_tensor(cfg["pos"] + move, device=dev))
    want = [(move[cfg["types"] == a] ** 2).sum(1).mean() for a in (0, 1)]
    assert np.allclose(ctx.rbsog_msd(), want, rtol=1e-12, atol=0)
    assert np.allclose(ctx.rbsog_msd(), want, rtol=1e-12, atol=0)
