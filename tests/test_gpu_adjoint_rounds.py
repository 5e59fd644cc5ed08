"""The adjoint step's local kernel on 64 x 8 tiles (FP32 lattices that they fill for one
or two rounds), and on 32 x 4 tiles of narrow lattices: a lattice periodic in y that is a
smaller one repeated stays its copies, bit for bit, the smaller one on other tiles.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _adjoint_step(case, k, seed):
    """(fbar, gbar, hbar) of one adjoint step on `case` repeated k times in y."""
    from paper_2111_00847_amd import api
    from paper_2111_00847_amd.sim import Sim
    rep = lambda a: np.concatenate([a] * k, axis=-2)
    phi0, u0, p0 = W.random_state_fields(case, seed=seed)
    big = case.replace(ny=k * case.ny)
    s = Sim(big).init(rep(phi0), rep(u0), rep(p0)).step(3)
    tape = api.new_tape(s.p, 1)
    api.lbm_tape_record(s.p, s.state, tape, 1)
    rng = np.random.default_rng(seed)
    dt = torch.float64 if case.dtype == "f64" else torch.float32
    bars = [torch.tensor(rep(rng.standard_normal((m, case.ny, case.nx))), dtype=dt, device="cuda") for m in (9, 9, 3)]
    adj = api.new_adjoint(s.p)
    api.lbm_adjoint_import(s.p, adj, *bars, 4)
    api.lbm_adjoint_step(s.p, tape, 0, adj)
    out = [torch.empty((m, big.ny, big.nx), dtype=dt, device="cuda") for m in (9, 9, 3)]
    api.lbm_adjoint_export(s.p, adj, *out)
    assert api.lbm_adjoint_params(s.p, adj)[1] == 3
    return out


SIZES = {(256, 250): 2, (250, 125): 4, (500, 125): 4, (20, 500): 8, (33, 1000): 4}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("wall_x", [False, True])
@pytest.mark.parametrize("size", list(SIZES), ids=[f"{a}x{b}x{k}" for (a, b), k in SIZES.items()])
def test_repeated_lattice_has_repeated_adjoints(size, wall_x, dtype):
    nx, ny = size
    case = W.Case(nx=nx, ny=ny, wall_x=wall_x, rhoA=20.0, nuA=0.05, nuB=0.2, sigma=0.01, M=0.05,
                  body_force=(1e-6, -2e-6), rho_ref=3.0, dtype=dtype, theta=(1.2, 1.9, 0.7, 2.4))
    small, big = _adjoint_step(case, 1, nx), _adjoint_step(case, SIZES[size], nx)
    for a, b in zip(small, big):
        for j in range(SIZES[size]):
            assert torch.equal(a, b[:, j * ny:(j + 1) * ny]), (size, j, float((a - b[:, j * ny:(j + 1) * ny]).abs().max()))
