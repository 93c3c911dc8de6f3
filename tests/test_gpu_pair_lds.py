"""Pair kernel launches whose tables and draw masks come near the 160 KB of LDS
of a workgroup: the workgroup takes fewer atoms then, or one lane an atom, and
the result keeps its bits."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
from force_bars import check_forces
from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


def _system(cfg, precision, **over):
    import torch
    dev = torch.device("cuda", 0)
    ctx = R.Context(0)
    ctx.rbsog_set_system(R.make_params(dict(cfg["sys"], p_f=20, **over), precision, n_atoms=len(cfg["types"])),
                         *(torch.as_tensor(cfg[k], device=dev) for k in ("types", "pos", "vel")))
    return ctx


def _forces(ctx):
    f, e = ctx.rbsog_compute_forces(3)
    g, _ = ctx.rbsog_compute_forces(3, want_energy=False)
    return f.cpu().numpy(), g.cpu().numpy(), e


@pytest.mark.parametrize("n,precision", [(33002, "fp64"), (70002, "mixed")])
def test_largest_capacity_with_every_workgroup(n, precision):
    """One lane an atom; the largest candidate capacity a caller may ask for."""
    print(f"case: capacity 4096 n {n} {precision}", flush=True)
    cfg = W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3))
    prec = R.FP64 if precision == "fp64" else R.MIXED
    ctx = _system(cfg, prec, p_r=20)
    ref = _forces(ctx)
    assert ctx.rbsog_set_list_capacity(128, 4096) == (128, 4096)
    for block in (64, 128, 256):
        ctx.rbsog_set_tuning(pair_block=block)
        assert ctx.rbsog_get_tuning()["pair_block"] == block
        got = _forces(ctx)
        np.testing.assert_array_equal(got[0], ref[0])
        np.testing.assert_array_equal(got[1], ref[1])
        assert dict(got[2], n_builds=0) == dict(ref[2], n_builds=0)
    assert ctx.rbsog_autotune(1)["pair_block"] in (64, 128, 256)
    np.testing.assert_array_equal(_forces(ctx)[0], ref[0])


def test_default_shape_at_a_long_cutoff():
    """A cutoff of 47 A: about 5100 candidates an atom (room for 7700, masks of
    60 KB per 64 atoms) and a table of twelve binades, with the shapes a set
    chooses."""
    print("case: r_shell 47", flush=True)
    cfg = W.config("nacl_512", n=33002, box=144.2)
    over = dict(r_shell=47.0, skin=1.0, p_r=20)
    ctx = _system(cfg, R.FP64, **over)
    f, g, _ = _forces(ctx)
    assert np.abs(f - g).max() <= 1e-12 * np.abs(f).max()
    short = ctx.rbsog_get_force_parts()[0].cpu().numpy()
    sel = np.sort(np.random.default_rng(1).choice(len(f), 100, replace=False)).astype(np.int32)
    fo = O.System(dict(cfg["sys"], p_f=20, **over), cfg["types"], cfg["pos"], cfg["vel"]).forces_short_atoms(3, sel)
    check_forces(short[sel], fo, 1e-11, "short-range force")
