"""The pair kernel with one to four lanes sharing an atom's lists.  The lane
count follows the size of the whole launch and must not change a bit: a small
system alone (four lanes) against itself in batches whose other system makes
the launch take fewer, over batch sizes at the edges of a
round of groups, of the drawn-together limit (64) and of take-all, odd ion
counts, both forms, stored batches and energies; and against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
from force_bars import check_forces
from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu

FILLERS = {"two fp64": 25_000, "some": 50_000, "one": 300_000}  # lanes FP64 2, 1, 1; mixed 4, 2, 1


def _cfg(n, seed=3):
    return W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3), melt_seed=seed)


@pytest.fixture(scope="module")
def fillers():
    return {k: _cfg(n, 11) for k, n in FILLERS.items()}


def _batch(cfgs, precision, want_energy, **over):
    import torch
    ctx = R.Context(0)
    dev = torch.device("cuda", 0)
    ctx.rbsog_set_batch([R.make_params(dict(c["sys"], p_f=20, **over), precision, n_atoms=len(c["types"]))
                         for c in cfgs],
                        *(torch.as_tensor(np.concatenate([c[k] for c in cfgs]), device=dev)
                          for k in ("types", "pos", "vel")))
    f, e = ctx.rbsog_compute_forces(4, want_energy=want_energy)
    fs, _ = ctx.rbsog_get_force_parts()
    n = len(cfgs[0]["types"])
    e = e[0] if isinstance(e, list) else e
    return f[:n].cpu().numpy(), fs[:n].cpu().numpy(), e


@pytest.mark.parametrize("stored", [False, True])
@pytest.mark.parametrize("precision", [R.FP64, R.MIXED])
@pytest.mark.parametrize("n,p_r", [(514, 1), (642, 20), (1000, 33), (514, 64), (514, 65), (642, 400), (642, 0)])
def test_lanes_do_not_change_a_bit(fillers, n, p_r, precision, stored):
    print(f"case: pair lanes n {n} p_r {p_r} precision {precision} stored {stored}", flush=True)
    if stored and p_r == 0:
        pytest.skip("a stored batch needs p_r >= 1")
    c = _cfg(n)
    alone = _batch([c], precision, True, p_r=p_r, shell_stored=stored)
    for lanes in FILLERS:
        got = _batch([c, fillers[lanes]], precision, True, p_r=p_r, shell_stored=stored)
        assert np.array_equal(alone[0], got[0]) and np.array_equal(alone[1], got[1]), lanes
        assert alone[2] == got[2], lanes
    plain = _batch([c], precision, False, p_r=p_r, shell_stored=stored)
    assert np.array_equal(alone[1], plain[1])
    sysp = dict(c["sys"], p_f=20, p_r=p_r, shell_stored=stored)
    osys = O.System(sysp, c["types"], c["pos"], c["vel"])
    osys.build_lists()
    fo, eo = osys.forces(4)
    tol = 1e-11 if precision == R.FP64 else 1e-5
    check_forces(alone[0], fo, tol, "force")
    for key in ("u_core", "u_shell", "virial", "stress", "heat_flux"):
        a, b = np.atleast_1d(alone[2][key]), np.atleast_1d(eo[key])
        assert np.abs(a - b).max() <= 10 * tol * max(np.abs(b).max(), 1e-30), key


def test_species_radii_and_orthorhombic_box_by_lanes(fillers):
    """Per-pair core radii and a box split along some axes only (the minimum
    image of every difference)."""
    print("case: pair lanes species radii", flush=True)
    c = _cfg(1000)
    rcp = [[5.5, 4.0], [4.0, 6.0]]
    alone = _batch([c], R.FP64, True, r_core_pair=rcp)
    got = _batch([c, fillers["one"]], R.FP64, True, r_core_pair=rcp)
    assert np.array_equal(alone[0], got[0]) and alone[2] == got[2]
