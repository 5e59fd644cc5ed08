"""Set-up and read-back calls on the sizes where their kernels change shape.

lbm_hydrostatic_pressure keeps column sums and the mean in the bytes of p0 and runs
the columns' chains over chunks of 256 rows, 16 columns to a workgroup: one node,
one row, one column, ragged columns, a ragged last chunk, a p0 that is phi0 itself.
Against the trapezoid integral in extended precision: a column's value is a chain
of ny additions, so FP64 is held to ny rounding errors of the largest partial
integral and FP32 to one rounding (of the result) more.

lbm_init, lbm_export_state and lbm_import_state: the exported state of a fresh
lattice carries the equilibrium's moments, and an imported state exports the same
bits, on lattices with every boundary kind, narrower than the stencil too.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("size", [(1, 1), (1, 2), (2, 1), (1, 300), (3, 2), (2, 2), (9, 127), (8, 129), (64, 32),
                                  (65, 63), (17, 256), (16, 257), (257, 1000)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_hydrostatic_pressure(size, dtype, in_place):
    from paper_2111_00847_amd import api
    nx, ny = size
    case = W.Case(nx=nx, ny=ny, rhoA=1000.0, gravity=(0.0, -1e-3), rho_ref=2.0, dtype=dtype)
    p = api.make_params(case)
    npt = np.float64 if dtype == "f64" else np.float32
    phi = np.random.default_rng(nx + ny).uniform(0.0, 1.0, (ny, nx)).astype(npt)
    t = torch.tensor(phi, device="cuda")
    out = t if in_place else torch.empty_like(t)
    api.lbm_hydrostatic_pressure(p, t, out)
    ld = np.longdouble
    f = (ld(999.0) * phi.astype(ld) + ld(1.0) - ld(2.0)) * ld(-1e-3)
    ref = np.zeros((ny, nx), dtype=ld)
    for j in range(ny - 2, -1, -1):
        ref[j] = ref[j + 1] - ld(0.5) * (f[j] + f[j + 1])
    scale = float(np.abs(ref).max()) or 1.0
    ref -= ref.mean()
    err = float(np.abs(out.cpu().numpy().astype(ld) - ref).max()) / scale
    tol = (ny + 10) * 1.2e-16 + (6.0e-8 if dtype == "f32" else 0.0)
    print(f"{size} {dtype} in_place={in_place}: {err:.2e} (bound {tol:.2e})", flush=True)
    assert err <= tol


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["stencil", "local", "cahn_hilliard"])
@pytest.mark.parametrize("size", [(1, 3, 0, 0), (2, 2, 1, 1), (3, 5, 0, 1), (4, 3, 1, 0), (70, 41, 1, 1), (300, 200, 0, 1)],
                         ids=lambda s: f"{s[0]}x{s[1]}")
def test_init_export_import(size, dtype, kind):
    from paper_2111_00847_amd.sim import Sim
    nx, ny, wx, wy = size
    kw = dict(phase_eq="cahn_hilliard", phiA=1.0, phiB=-1.0) if kind == "cahn_hilliard" else {}
    case = W.Case(nx=nx, ny=ny, wall_x=bool(wx), wall_y=bool(wy), rhoA=20.0, sigma=0.01, M=0.05, dtype=dtype,
                  theta=(1.2, 1.9, 0.7, 2.4), grad_scheme="local" if kind == "local" else "stencil", **kw)
    phi0, u0, p0 = W.random_state_fields(case, seed=3)
    sim = Sim(case).init(phi0, u0, p0)
    d = sim.export_state()
    assert d["step"] == 0 and float(d["hist"].abs().max()) == 0.0
    tol = 1e-12 if dtype == "f64" else 2e-5
    phi = d["f"].double().sum(0).cpu().numpy()
    assert np.abs(phi - phi0).max() <= tol
    assert np.abs(d["g"].double().sum(0).cpu().numpy()).max() <= tol * max(1.0, float(d["g"].abs().max()))   # rho0 = 0
    hist = torch.rand_like(d["hist"])
    e = Sim(case).import_state(d["f"], d["g"], hist, 7).export_state()
    assert e["step"] == 7 and torch.equal(e["hist"], hist) and torch.equal(e["g"], d["g"])
    assert torch.equal(e["f"][1:], d["f"][1:])
    # f_0 is stored relative to the history phi: one rounding of its type
    assert float((e["f"][0] - d["f"][0]).abs().max()) <= (0.0 if dtype == "f64" else 1.2e-7)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("size", [(1023, 40), (1025, 20), (2000, 300), (4100, 33)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_hydrostatic_pressure_in_place_has_the_same_bits(size, dtype):
    """A p0 that is phi0 itself runs in one workgroup, another array in staged
    columns: the same additions in the same order, the mean's included (wider
    than its 1024 threads too), so the same bits."""
    from paper_2111_00847_amd import api
    nx, ny = size
    p = api.make_params(W.Case(nx=nx, ny=ny, rhoA=1000.0, gravity=(0.0, -1e-3), rho_ref=2.0, dtype=dtype))
    gen = torch.Generator().manual_seed(nx)
    t = torch.rand((ny, nx), generator=gen, dtype=torch.float64).to("cuda", torch.float64 if dtype == "f64" else torch.float32)
    out = torch.empty_like(t)
    api.lbm_hydrostatic_pressure(p, t, out)
    api.lbm_hydrostatic_pressure(p, t, t)
    assert torch.equal(out, t), float((out - t).abs().max())
