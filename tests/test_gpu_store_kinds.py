"""Two-level launches by store kind: batches and tapes whose rows end inside a
cache line, and whose rows do not, against one-level launches bit for bit.

Which stores a launch uses follows the bytes of the state (written through the
L2 while the last-level cache holds it, else non-temporal) and whether rows are
whole 128-byte lines (ordinary stores where they are not).
"""
import os

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(nx, ny, dtype):
    return W.Case(nx=nx, ny=ny, wall_x=nx % 4 == 2, wall_y=ny % 2 == 0, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01,
                  M=0.05, gravity=(0.0, -1e-5), rho_ref=3.0, dtype=dtype, theta=(1.2, 1.9, 0.7, 2.4))


BATCHES = {   # sizes of the cases -> how the batch is stored (FP32; FP64 twice the bytes)
    "broken rows, above a third of the cache": [(500, 300)] * 4 + [(131, 75)],
    "broken rows, streamed": [(1001, 700)] * 3 + [(67, 41)],
    "one case of broken rows": [(512, 384)] * 4 + [(33, 40)],
    "whole rows, streamed": [(1024, 700)] * 3 + [(64, 41)],
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", list(BATCHES))
def test_batch_equals_lone_one_level_runs(kind, dtype):
    from paper_2111_00847_amd import api
    from paper_2111_00847_amd.sim import BatchSim, Sim
    cases = [_case(nx, ny, dtype) for nx, ny in BATCHES[kind]]
    phis = [W.random_state_fields(c, seed=k)[0] for k, c in enumerate(cases)]
    print(kind, dtype, flush=True)
    a, b = BatchSim(cases).init(phis), BatchSim(cases).init(phis)
    a.step(5)
    api.lbm_batch_step_noalloc(b.params, b.state, 5)
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        for k, c in enumerate(cases):
            want = Sim(c).init(phis[k]).step(5).export_state()
            for batch in (a, b):
                got = batch.case(k).export_state()
                assert got["step"] == 5
                for q in ("f", "g", "hist"):
                    assert torch.equal(got[q], want[q]), (k, q)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)


TAPES = {   # size -> the tile shape the rule takes there (FP32 / FP64)
    (125, 60): "16x4", (250, 126): "32x4", (250, 250): "32x8, one round", (256, 250): "32x8, one round, whole rows",
    (250, 500): "32x16, one round", (250, 1020): "64x16 / 32x8", (256, 1020): "64x16 / 32x8, whole rows",
    (1020, 500): "32x16 / 32x8", (1024, 500): "32x16 / 32x8, whole rows", (1020, 700): "64x8 / 32x8",
    (2050, 1100): "64x8 / 32x8, streamed", (2048, 1100): "64x8 / 32x8, streamed, whole rows",
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("size", list(TAPES), ids=[f"{a}x{b}" for a, b in TAPES])
def test_tape_slots_equal_one_level_launches(size, dtype):
    """Every slot of a tape -- those between two launches, those a launch stores
    on its way, and the last one of an odd count -- holds the level that
    one-level launches give."""
    from paper_2111_00847_amd import api
    from paper_2111_00847_amd.sim import Sim
    nx, ny = size
    case = _case(nx, ny, dtype)
    phi0, u0, p0 = W.random_state_fields(case, seed=nx + ny)
    print(f"tape {nx}x{ny} {dtype}: {TAPES[size]}", flush=True)
    a, b, c = (Sim(case).init(phi0, u0, p0) for _ in range(3))
    slots = 6
    tape = api.new_tape(a.p, slots)
    api.lbm_tape_record(a.p, a.state, tape, slots)
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        for j in range(slots):
            api.lbm_tape_restore(a.p, tape, j, c.state)
            got, want = c.export_state(), b.export_state()
            assert got["step"] == want["step"] == j
            for k in ("f", "g", "hist"):
                assert torch.equal(got[k], want[k]), (j, k)
            b.step(1)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)
