"""lbm_export_state and lbm_import_state on large lattices: FP64 states exported population
by population (more than 256 MB written), and copies beyond 4 GiB in either type.  A lattice
that is a small one repeated in x exports the small one's state repeated, bit for bit, and
exports again what it imports.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,nx,ny,k", [("f64", 130, 1301, 10), ("f64", 256, 1024, 100), ("f32", 256, 1024, 200)])
def test_export_of_a_repeated_lattice(dtype, nx, ny, k):
    from paper_2111_00847_amd.sim import Sim
    case = W.Case(nx=nx, ny=ny, rhoA=20.0, sigma=0.01, M=0.05, dtype=dtype)
    phi0, u0, p0 = W.random_state_fields(case, seed=5)
    a = Sim(case).init(phi0, u0, p0).step(3).export_state()
    big = case.replace(nx=k * nx)
    rep = lambda t: t.repeat(1, 1, k)
    sim = Sim(big).init(*(np.concatenate([x] * k, axis=-1) for x in (phi0, u0, p0))).step(3)
    for e in (sim.export_state(), Sim(big).import_state(rep(a["f"]), rep(a["g"]), rep(a["hist"]), a["step"]).export_state()):
        assert e["step"] == 3
        for name in ("f", "g", "hist"):
            assert torch.equal(e[name], rep(a[name])), name
        del e
    torch.cuda.empty_cache()
