"""lbm_levels_per_launch never reports more levels than a launch advances."""
import ctypes
import os

import pytest

import workloads as W


def _levels(**kw):
    from paper_2111_00847_amd import _lib, api
    v = ctypes.c_int32(-1)
    p = api.make_params(W.Case(rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05, **kw))
    assert ctypes.CDLL(_lib.LIB_PATH).lbm_levels_per_launch(ctypes.byref(p), ctypes.byref(v)) == 0
    return v.value


@pytest.mark.parametrize("mode", [None, "1"])
def test_one_row_in_fp64_runs_one_level(mode):
    """FP64 lattices of one row have fewer level stamps than tiles and run one level
    per launch, whatever their length; FP32 ones run two."""
    if mode is None:
        os.environ.pop("LBM_TWO_LEVEL", None)
    else:
        os.environ["LBM_TWO_LEVEL"] = mode
    try:
        for nx in (17000, 60000):
            assert _levels(nx=nx, ny=1, dtype="f64") == 1
            assert _levels(nx=nx, ny=1, dtype="f32") == 2
            assert _levels(nx=nx, ny=2, dtype="f64") == 2
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_batch_with_one_row(dtype):
    from paper_2111_00847_amd.sim import BatchSim
    cases = [W.Case(nx=nx, ny=ny, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05, dtype=dtype)
             for nx, ny in ((20000, 1), (128, 64))]
    assert BatchSim(cases).levels_per_launch() == (2 if dtype == "f32" else 1)
    assert BatchSim([cases[1].replace(nx=1024, ny=512)]).levels_per_launch() == 2


@pytest.mark.gpu
def test_two_level_switch_is_read_at_every_call():
    """LBM_TWO_LEVEL=0 also stops two-level launches where a graph of them is
    cached: after one-level launches the other copy of the state holds the level
    before the last (after two-level ones, the level two before it)."""
    import torch
    from paper_2111_00847_amd.sim import Sim
    case, phi0 = W.square_droplet(n=64, side=32)
    s = torch.cuda.Stream()
    a, b = Sim(case, stream=s).init(phi0), Sim(case, stream=s).init(phi0)
    torch.cuda.synchronize()
    b.state.copy_(a.state)
    torch.cuda.synchronize()
    a.step(64)                # captures and replays a graph of two-level launches
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        b.step(64)
        a.step(64)
        b.step(64)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)
    torch.cuda.synchronize()
    assert torch.equal(a.state, b.state)
