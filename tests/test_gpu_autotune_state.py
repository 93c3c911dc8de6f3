"""Tuning leaves the state as it was: a run tuned between two step calls, or
after new positions, goes on bit for bit as one that was not, with no force
evaluation of the caller's in between.  Small systems (one stream) and one whose
k-space chain runs on the second stream."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(cfg, precision, tune, moved):
    import torch
    dev = torch.device("cuda", 0)
    ctx = R.Context(0)
    ctx.rbsog_set_system(R.make_params(dict(cfg["sys"], p_f=40, t_target=1200.0, tau_t=0.01), precision,
                                       n_atoms=len(cfg["types"])),
                         *(torch.as_tensor(cfg[k], device=dev) for k in ("types", "pos", "vel")))
    ctx.rbsog_step(4)
    if moved:  # no forces at the new positions yet
        ctx.rbsog_set_positions(ctx.rbsog_get_state()[0] + 0.01)
    if tune:
        ctx.rbsog_autotune(1)
    out = [] if moved else [x.cpu().numpy() for x in ctx.rbsog_get_state()[:3]]
    if not moved:
        out += [x.cpu().numpy() for x in ctx.rbsog_get_force_parts()] + [ctx.rbsog_get_rho(40)]
    e = ctx.rbsog_step(5)
    out += [x.cpu().numpy() for x in ctx.rbsog_get_state()[:3]]
    ctx.close()
    return out, e


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,moved", [(512, False), (2050, True), (140002, False)])
def test_tuning_leaves_the_state(n, moved, precision):
    print(f"case: n {n} moved {moved} {precision}", flush=True)
    prec = R.FP64 if precision == "fp64" else R.MIXED
    cfg = W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3), melt_seed=7)
    a, ea = _run(cfg, prec, False, moved)
    b, eb = _run(cfg, prec, True, moved)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)
    assert ea["u_total"] == eb["u_total"] and ea["kinetic"] == eb["kinetic"]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,p_f,fixed", [(512, 100, ("pair_block", "pair_ku", "kf_block", "kf_aux")),
                                         (100002, 20, ("kf_aux",))])
def test_tuning_keeps_values_without_effect(n, p_f, fixed, precision):
    """Several lanes an atom and shared modes have launch shapes of their own,
    and one stream (up to 131072 ions) has no place of the k-space force to
    choose: whatever the tuner times, those values stay as they were set."""
    import torch
    print(f"case: values without effect n {n} {precision}", flush=True)
    cfg = W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3), melt_seed=7)
    dev = torch.device("cuda", 0)
    ctx = R.Context(0)
    ctx.rbsog_set_system(R.make_params(dict(cfg["sys"], p_f=p_f), R.FP64 if precision == "fp64" else R.MIXED, n_atoms=n),
                         *(torch.as_tensor(cfg[k], device=dev) for k in ("types", "pos", "vel")))
    for over in (dict(pair_block=256, pair_ku=8, kf_block=64, kf_aux=0),
                 dict(pair_block=128, pair_ku=4, kf_block=128, kf_aux=1)):
        ctx.rbsog_set_tuning(**over)
        got = ctx.rbsog_autotune(1)
        assert got == ctx.rbsog_get_tuning()
        for key in fixed:
            assert got[key] == over[key], (key, got)
