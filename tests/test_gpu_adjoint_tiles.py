"""The tile shapes of the adjoint step's local kernel: 32 x 4 on small lattices
(the other adjoint tests), 64 x 4 where those would be more than two to a CU.

One FP64 adjoint step on lattices of either side of that line (ragged in both
directions) equals the autograd vector-Jacobian product of one reference step,
element by element, to 1e-11 of the largest entry (the tolerance of the small
lattices: the same arithmetic per node).
"""
import numpy as np
import pytest

from test_gpu_adjoint import GEOMS, _api, _case, _close, _random_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("size", [(255, 250), (291, 230), (66, 1021)], ids=["32x4", "64x4", "64x4_tall"])
@pytest.mark.parametrize("geom", list(GEOMS))
def test_one_adjoint_step_equals_reference_vjp(size, geom):
    from oracle.torch_ref import TorchRef, as_params
    api, Sim = _api()
    n = 4
    case = _case(geom, *size)
    f, g, php, upr = _random_state(case, seed=11)
    s = Sim(case).import_state(f, g, np.concatenate([php[None], upr], 0), n)
    tape = api.new_tape(s.p, 1)
    api.lbm_tape_record(s.p, s.state, tape, 1)
    rng = np.random.default_rng(12)
    shp = (case.ny, case.nx)
    bars = [rng.standard_normal((k,) + shp) for k in (9, 9, 3)]
    adj = api.new_adjoint(s.p)
    api.lbm_adjoint_import(s.p, adj, *[torch.tensor(b, device="cuda") for b in bars], n + 1)
    api.lbm_adjoint_step(s.p, tape, 0, adj)
    out = [torch.empty((k,) + shp, dtype=torch.float64, device="cuda") for k in (9, 9, 3)]
    api.lbm_adjoint_export(s.p, adj, *out)
    prm, level = api.lbm_adjoint_params(s.p, adj)
    assert level == n
    ref = TorchRef(case)
    grav, theta = as_params(case)
    st = dict(f=torch.tensor(f, requires_grad=True), g=torch.tensor(g, requires_grad=True),
              phi_prev=torch.tensor(php, requires_grad=True), u_prev=torch.tensor(upr, requires_grad=True), n=n)
    r = ref.step(st, grav, theta)
    ((r["f"] * torch.tensor(bars[0])).sum() + (r["g"] * torch.tensor(bars[1])).sum() +
     (r["phi_prev"] * torch.tensor(bars[2][0])).sum() + (r["u_prev"] * torch.tensor(bars[2][1:])).sum()).backward()
    tag = f"{size} {geom}"
    _close(out[0].cpu().numpy(), st["f"].grad.numpy(), 1e-11, tag + " fbar")
    _close(out[1].cpu().numpy(), st["g"].grad.numpy(), 1e-11, tag + " gbar")
    _close(out[2][0].cpu().numpy(), st["phi_prev"].grad.numpy(), 1e-11, tag + " phi_prev bar")
    _close(out[2][1:].cpu().numpy(), st["u_prev"].grad.numpy(), 1e-11, tag + " u_prev bar")
    _close(prm[0:2], grav.grad.numpy(), 1e-10, tag + " dgravity")
    if geom != "periodic":
        _close(prm[2:6], theta.grad.numpy(), 1e-10, tag + " dtheta")
