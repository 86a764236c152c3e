"""The reverse step's reduction of its parameter gradients: fewer block partials
than threads, whole batches of loads, batches cut short, and blocks of one wave
and of four (up to and beyond 65536 sites), against autograd through the oracle's
torch transcription of the step."""
from __future__ import annotations

import pytest
import torch

import lbinputs
import oracle.reverse as R
from _gpu import rel_err

pytestmark = pytest.mark.gpu


# FP32 storage: the gradients are within 5e-6 - 3e-5 of the FP64 adjoint's over
# rollouts of up to 1000 steps; 2 steps round far less
@pytest.mark.parametrize("shape,prec,tol", [((3, 5, 4), "fp64", 1e-10),
                                            ((16, 16, 16), "fp64", 1e-10),
                                            ((16, 16, 17), "fp64", 1e-10),
                                            ((32, 32, 32), "fp64", 1e-10),
                                            ((33, 32, 32), "fp64", 1e-10),
                                            ((40, 40, 40), "fp64", 1e-10),
                                            ((41, 40, 40), "fp64", 1e-10),
                                            ((16, 16, 17), "fp32_dev", 3e-5),
                                            ((25, 29, 28), "fp32_dev", 3e-5)])
@pytest.mark.parametrize("coupling", ["stress", "force"])
@pytest.mark.parametrize("order_param,tau_g", [("lb", 1.3), ("lb", 1.0), ("fd", 1.3)])
def test_adjoint_matches_oracle(order_param, tau_g, coupling, shape, prec, tol):
    from paper_1609_01479_amd.rollout import rollout
    T = 2
    pr = dict(lbinputs.SPINODAL_PARAMS, tau_f=0.8, tau_g=tau_g)
    phi0 = lbinputs.spinodal_phi0(shape, seed=31, amp=0.3)
    tgt = lbinputs.lamellar_target(shape, 8, lbinputs.interface_width(pr["A"], pr["kappa"]))
    print(f"[adjoint blocks] {shape} {prec} {order_param} {coupling} tau_g={tau_g}", flush=True)
    dev = torch.device("cuda:0")
    p0 = torch.tensor(phi0, dtype=torch.float64, device=dev, requires_grad=True)
    th = [torch.tensor(pr[k], dtype=torch.float64, device=dev, requires_grad=True)
          for k in ("A", "B", "kappa")]
    phiT = rollout(p0, *th, T, interval=2, gamma=pr["gamma"], tau_f=pr["tau_f"],
                   tau_g=pr["tau_g"], rho0=pr["rho0"], order_param=order_param,
                   coupling=coupling, precision=prec)
    loss = 0.5 * ((phiT - torch.tensor(tgt, device=dev)) ** 2).sum()
    grads = torch.autograd.grad(loss, [p0] + th)
    fn = R.fd_loss_and_grads if order_param == "fd" else R.loss_and_grads
    _, rphi, *rth = fn(phi0, tgt, pr["A"], pr["B"], pr["kappa"], T, pr["gamma"], pr["tau_f"],
                       pr["tau_g"], pr["rho0"], coupling)
    err = rel_err(grads[0].cpu().numpy(), rphi)
    assert err <= tol, err
    for name, t, b in zip(("A", "B", "kappa"), grads[1:], rth):
        assert abs(float(t) - b) <= 10 * tol * abs(b), (name, float(t), b)
