"""Two-level launches on lattices of few rows, at the edges of the rule that keeps
tiles of 16 rows off them, against one-level launches bit for bit."""
import os

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("size", [(17000, 2), (9000, 8), (9000, 9), (17000, 17), (9000, 40), (7000, 48), (9000, 49)],
                         ids=lambda s: f"{s[0]}x{s[1]}")
def test_flat_lattice_equals_one_level_launches(size, dtype):
    from paper_2111_00847_amd.sim import Sim
    nx, ny = size
    case = W.Case(nx=nx, ny=ny, wall_y=ny % 2 == 1, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05,
                  gravity=(0.0, -1e-5), rho_ref=3.0, dtype=dtype, theta=(1.2, 1.9, 0.7, 2.4))
    phi0, u0, p0 = W.random_state_fields(case, seed=ny)
    a, b = Sim(case).init(phi0, u0, p0), Sim(case).init(phi0, u0, p0)
    a.step(5)
    os.environ["LBM_TWO_LEVEL"] = "0"
    try:
        b.step(5)
    finally:
        os.environ.pop("LBM_TWO_LEVEL", None)
    sa, sb = a.export_state(), b.export_state()
    assert sa["step"] == sb["step"] == 5
    for k in ("f", "g", "hist"):
        assert torch.equal(sa[k], sb[k]), (k, float((sa[k] - sb[k]).abs().max()))
