"""Steps cut into calls: a call that follows a step takes over the velocity
factor which that step left, and any other call forms it from the velocities
again.  Both are sums of the same terms in the same order, so however a run is
cut the state has the same bits; Nose-Hoover, whose factor at a call's start is
rounded once more, agrees to rounding grown over nine steps.  Snapshots, taken at
every call, are exercised by odd counts (ends not aligned to 16 bytes)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(cfg, precision, cuts, **over):
    import torch
    ctx = R.Context(0)
    dev = torch.device("cuda", 0)
    ctx.rbsog_set_system(R.make_params(dict(cfg["sys"], p_f=20, **over), precision, n_atoms=len(cfg["types"])),
                         *(torch.as_tensor(cfg[k], device=dev) for k in ("types", "pos", "vel")))
    for k, c in enumerate(cuts):
        e = ctx.rbsog_step(c, want_energy=k == len(cuts) - 1)
    out = [x.cpu().numpy() for x in ctx.rbsog_get_state()[:3]]
    ctx.close()
    return out, e


@pytest.mark.parametrize("n", [216, 2502])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("thermostat", ["berendsen", "langevin", "nose_hoover"])
def test_state_does_not_depend_on_the_calls(n, precision, thermostat):
    print(f"case: n {n} {precision} {thermostat}", flush=True)
    prec = R.FP64 if precision == "fp64" else R.MIXED
    cfg = W.config("nacl_small", n=n, box=(n / 0.0191) ** (1 / 3))
    over = dict(t_target=1000.0, tau_t=0.02, thermostat=thermostat)
    whole, ew = _run(cfg, prec, [9], **over)
    for cuts in ([3, 1, 5], [8, 1]):
        got, eg = _run(cfg, prec, cuts, **over)
        if thermostat != "nose_hoover":
            for a, b in zip(whole, got):
                np.testing.assert_array_equal(a, b)
            assert eg["kinetic"] == ew["kinetic"]
        elif prec == R.FP64:
            for a, b in zip(whole, got):
                np.testing.assert_allclose(a, b, rtol=0, atol=1e-9 * np.abs(a).max())
