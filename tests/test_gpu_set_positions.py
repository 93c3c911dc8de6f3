"""rbsog_set_positions from every kind of memory it takes: this device's memory
read in place, on the default and on another stream, and the buffers the
runtime copies first (host memory, a pointer that is not a multiple of eight
bytes).  All give the same bits; a refused call changes nothing."""
from __future__ import annotations

import ctypes as C

import numpy as np
import pytest

from paper_2512_24970_amd import rbsog as R
from paper_2512_24970_amd import workloads as W

pytestmark = pytest.mark.gpu


def _batch(stream=None):
    import torch
    cfgs = [W.config("nacl_512", n=n, box=(n / 0.0319) ** (1 / 3), replica=r, melt_seed=5 + r)
            for r, n in enumerate((514, 1000, 642))]
    dev = torch.device("cuda", 0)
    ctx = R.Context(0, stream=stream)
    cat = lambda k: torch.as_tensor(np.concatenate([c[k] for c in cfgs]), device=dev)
    torch.cuda.synchronize()
    ctx.rbsog_set_batch([R.make_params(c["sys"], R.MIXED, n_atoms=len(c["types"])) for c in cfgs],
                        cat("types"), cat("pos"), cat("vel"))
    return ctx, np.concatenate([c["pos"] for c in cfgs])


def _state(ctx):
    import torch
    f, e = ctx.rbsog_compute_forces(3)
    pos = ctx.rbsog_get_state()[0]
    torch.cuda.synchronize()
    return pos.cpu().numpy(), f.cpu().numpy(), [x["max_disp"] for x in e], [x["u_total"] for x in e]


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("route", ["device", "stream", "host", "unaligned"])
def test_every_route_gives_the_same_bits(route):
    import torch
    print(f"case: set_positions {route}", flush=True)
    ref, pos0 = _batch()
    pos = pos0 + np.random.default_rng(8).uniform(-0.2, 0.2, pos0.shape)
    ref.rbsog_set_positions(torch.as_tensor(pos, device="cuda"))
    ctx, _ = _batch(torch.cuda.Stream() if route == "stream" else None)
    if route in ("device", "stream"):
        ctx.rbsog_set_positions(torch.as_tensor(pos, device="cuda") * 1.0)
    elif route == "host":
        assert R.lib().rbsog_set_positions(ctx._h, C.c_void_p(np.ascontiguousarray(pos).ctypes.data), 0) == 0
    else:
        raw = torch.zeros(pos.nbytes + 8, dtype=torch.uint8, device="cuda")
        raw[4:4 + pos.nbytes] = torch.as_tensor(np.ascontiguousarray(pos).view(np.uint8).reshape(-1), device="cuda")
        torch.cuda.synchronize()
        assert R.lib().rbsog_set_positions(ctx._h, C.c_void_p(raw.data_ptr() + 4), 1) == 0
    a, b = _state(ref), _state(ctx)
    assert _same(a, b)
    assert 0.2 < max(a[2]) < 0.35


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("row", [0, 513, 2155])
def test_refused_positions_change_nothing(row, value):
    import torch
    print(f"case: refused positions row {row} {value}", flush=True)
    ctx, pos0 = _batch()
    pos = pos0 + np.random.default_rng(9).uniform(-0.2, 0.2, pos0.shape)
    ctx.rbsog_set_positions(torch.as_tensor(pos, device="cuda"))
    before = _state(ctx)
    bad = pos0.copy()
    bad[row, row % 3] = value
    with pytest.raises(R.RbsogError) as e:
        ctx.rbsog_set_positions(torch.as_tensor(bad, device="cuda"))
    assert e.value.code == -8
    assert _same(before, _state(ctx))
    ctx.rbsog_set_positions(torch.as_tensor(pos0, device="cuda"))
    assert max(_state(ctx)[2]) < 1e-9
