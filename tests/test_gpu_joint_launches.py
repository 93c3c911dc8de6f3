"""Small launches on one stream draw the modes beside the cell sort, sum the
structure factors beside the pair kernel and finalize them beside the force
sums.  Phase timing launches every kernel by itself, so a run with it is the
reference: the same blocks do the same work and the state must have the same
bits, over both lane counts, one lane (not joint), mode counts around a tile and
past the joint limit, the full sum, a batch, a stored batch and fixed-point phases (not joint),
launched one by one and from graphs."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(cfgs, precision, timed, graph, over):
    import torch
    dev = torch.device("cuda", 0)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = R.Context(0)
        ctx.rbsog_set_batch([R.make_params(dict(c["sys"], **over), precision, n_atoms=len(c["types"])) for c in cfgs],
                            *(torch.as_tensor(np.concatenate([c[k] for c in cfgs]), device=dev)
                              for k in ("types", "pos", "vel")))
        ctx.rbsog_profile_enable(timed)
        f0, _ = ctx.rbsog_compute_forces(3, want_energy=False)
        if graph:
            ctx.rbsog_step_batch(12)
            e = None
        else:
            ctx.rbsog_step(12, want_energy=False)
            e = ctx.rbsog_step(1)
        out = [x.cpu().numpy() for x in (f0, *ctx.rbsog_get_state()[:3])]
        ctx.close()
    return out, e


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,p_f,over", [
    ([512], 1, {}), ([514], 64, {}), ([2050], 65, {}), ([24002], 130, {}), ([40002], 64, {}), ([70002], 33, {}),
    ([16386], 2100, {}), ([514], 0, {}), ([512, 1500, 642], 100, {}), ([1500], 70, dict(shell_stored=True)),
    ([1500], 70, dict(int_phase=True)),
])
def test_joint_launches_change_no_bit(sizes, p_f, over, precision):
    if over.get("int_phase") and precision == "fp64":
        pytest.skip("fixed-point phases are the mixed form's")
    print(f"case: {sizes} p_f {p_f} {over} {precision}", flush=True)
    prec = R.FP64 if precision == "fp64" else R.MIXED
    cfgs = [W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3), melt_seed=5) for n in sizes]
    over = dict(over, p_f=p_f, t_target=1200.0, tau_t=0.01)
    for graph in (False, True):
        a, ea = _run(cfgs, prec, True, graph, over)
        b, eb = _run(cfgs, prec, False, graph, over)
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
        assert ea == eb
