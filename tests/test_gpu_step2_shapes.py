"""The tile shapes of the two-level launch, each where the size rule takes it.

lbm_step advances two levels per launch with the tile shape its size rule picks
(16 x 4 to 64 x 16 nodes).  Every shape runs here on a lattice of its own range,
ragged in both directions where the shape allows it, from level 0 and on: six
levels by one call equal six one-level launches (LBM_TWO_LEVEL=0) bit for bit.
The lattice of one row has fewer level stamps than tiles in FP64 and keeps
one-level launches.
"""
import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {   # size -> the shape the rule takes there (FP32 / FP64)
    (125, 60): "16x4", (64, 41): "32x4 (too few stamps for 16x4)", (250, 126): "32x4", (250, 250): "32x8, one round",
    (250, 500): "32x16, one round", (250, 1020): "64x16 / 32x8", (1020, 500): "32x16 cached / 32x8",
    (1020, 700): "64x8 cached / 32x8", (2050, 1100): "64x8 streamed / 32x8", (17000, 1): "64x8 / one level",
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("size", list(SHAPES), ids=[f"{a}x{b}" for a, b in SHAPES])
@pytest.mark.parametrize("grad", ["stencil", "local"])
def test_shape_equals_one_level_launches(size, dtype, grad):
    from paper_2111_00847_amd.sim import Sim
    nx, ny = size
    case = W.Case(nx=nx, ny=ny, wall_x=nx % 4 == 2, wall_y=ny > 1 and ny % 4 != 1, rhoA=20.0, nuA=0.05, nuB=0.2,
                  sigma=0.01, M=0.05, gravity=(0.0, -1e-5), rho_ref=3.0, dtype=dtype, theta=(1.2, 1.9, 0.7, 2.4),
                  grad_scheme=grad)
    phi0, u0, p0 = W.random_state_fields(case, seed=nx + ny)
    a, b = Sim(case).init(phi0, u0, p0), Sim(case).init(phi0, u0, p0)
    print(f"{nx}x{ny} {dtype} {grad}: {SHAPES[size]}", flush=True)
    a.step(6)
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        b.step(6)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)
    sa, sb = a.export_state(), b.export_state()
    assert sa["step"] == sb["step"] == 6
    for k in ("f", "g", "hist"):
        assert torch.equal(sa[k], sb[k]), (k, float((sa[k] - sb[k]).abs().max()))


BATCHES = {   # sizes of the cases -> the shape the rule takes for the batch
    "16x4": [(40, 32), (64, 64), (70, 40)], "32x4 (a case short of stamps)": [(61, 9), (128, 64), (40, 33)],
    "32x8, one round": [(256, 120), (130, 75)], "32x16, one round": [(250, 250), (130, 75), (5, 8)],
    "32x8": [(512, 256)] * 3 + [(130, 75), (2, 2)], "32x8 streamed": [(1024, 1024), (900, 1030), (37, 41)],
    "64x8 / one level": [(17000, 1), (70, 9)],
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", list(BATCHES))
def test_batch_shape_equals_lone_one_level_runs(shape, dtype):
    """Every case of a batch, seven levels on (an odd tail), against lone one-level
    runs; and the allocation-free step, which writes its own tables."""
    from paper_2111_00847_amd import api
    from paper_2111_00847_amd.sim import BatchSim, Sim
    cases = [W.Case(nx=nx, ny=ny, wall_y=ny > 1, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05, dtype=dtype,
                    theta=(1.2, 1.9, 0.7, 2.4)) for nx, ny in BATCHES[shape]]
    phis = [W.random_state_fields(c, seed=k)[0] for k, c in enumerate(cases)]
    print(shape, dtype, flush=True)
    a, b = BatchSim(cases).init(phis), BatchSim(cases).init(phis)
    a.step(7)
    api.lbm_batch_step_noalloc(b.params, b.state, 7)
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        for k, c in enumerate(cases):
            want = Sim(c).init(phis[k]).step(7).export_state()
            for batch in (a, b):
                got = batch.case(k).export_state()
                assert got["step"] == 7
                for q in ("f", "g", "hist"):
                    assert torch.equal(got[q], want[q]), (k, q)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)


MODELS = {"stencil": {}, "local": {"grad_scheme": "local"}, "corrected": {"model": "corrected"}, "ch": {}}


@pytest.mark.parametrize("size", [(2050, 400, 3, "f32"), (2048, 400, 3, "f32"), (1030, 400, 3, "f64"), (1024, 400, 3, "f64")],
                         ids=lambda s: f"{s[0]}x{s[1]}x{s[2]}_{s[3]}")
@pytest.mark.parametrize("model", list(MODELS))
def test_streamed_state_equals_its_cached_period(model, size):
    """A periodic lattice that is a smaller one repeated in y stays its copies, bit
    for bit: the smaller state fits the last-level cache (written through, swept
    forward), the larger one is streamed (swept forward and back by turns, stored
    non-temporally where its rows are whole cache lines).  Five levels in one call,
    then one, then two, so that launches of one and of two levels run both ways."""
    from paper_2111_00847_amd.sim import Sim
    nx, ny, k, dtype = size
    case = W.Case(nx=nx, ny=ny, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05, body_force=(1e-6, -2e-6),
                  rho_ref=3.0, dtype=dtype, **MODELS[model])
    phi0, u0, p0 = W.random_state_fields(case, seed=nx)
    if model == "ch":
        case, phi0 = W.to_cahn_hilliard(case, phi0)
    big = case.replace(ny=k * ny)
    rep = lambda a: np.concatenate([a] * k, axis=-2)
    a, b = Sim(case).init(phi0, u0, p0), Sim(big).init(rep(phi0), rep(u0), rep(p0))
    for n in (5, 1, 2):
        a.step(n)
        b.step(n)
        sa, sb = a.export_state(), b.export_state()
        for name in ("f", "g", "hist"):
            for i in range(k):
                assert torch.equal(sa[name], sb[name][:, i * ny:(i + 1) * ny]), (name, n, i)
