"""Training loops of the paper's QPINN on the circuit engine (section "PINN architecture and
convergence enhancements": Adam, learning rate 1e-3 decayed by 0.85 every 2000 epochs; the
total loss of eq. 2D_lossTot), timed per epoch like the paper's runtime table, and the black-hole
diagnostics (section "'Black hole' loss landscape").

* train_circuit: the circuit alone is the model (its first three readouts are the fields); each
  epoch is one qp_total_loss (or qp_maxwell_fused) call and an Adam step on the parameters.
* train_hybrid: the hybrid model of paper_2506_23246_amd.hybrid (classical network, circuit,
  linear head); the loss terms are formed in torch from the model's fields and their derivatives,
  and torch autograd runs the backward pass through the engine's adjoint.
"""
from __future__ import annotations

import time
from dataclasses import dataclass, field

import torch

from .hybrid import HybridQPINN, maxwell_residual_loss


@dataclass
class TrainLog:
    loss: list = field(default_factory=list)          # total loss per epoch
    terms: list = field(default_factory=list)         # (phys, ic, sym, energy) per epoch
    seconds: list = field(default_factory=list)       # wall time per epoch (stream synchronised)

    def s_per_epoch(self, skip: int = 1) -> float:
        s = self.seconds[skip:] if len(self.seconds) > skip else self.seconds
        return float(sum(s) / max(len(s), 1))


def _scheduler(opt, step=2000, gamma=0.85):
    return torch.optim.lr_scheduler.StepLR(opt, step_size=step, gamma=gamma)


def train_circuit(circuit, params, points, ic_xy, desc, epochs: int, lr: float = 1e-3, total: bool = True) -> TrainLog:
    """Adam on the circuit parameters with the library's gradient: qp_total_loss (total=True) or the
    residual loss alone (qp_maxwell_fused).  `circuit` is a compiled api.Circuit."""
    dev = circuit.ctx.dev
    p = torch.nn.Parameter(torch.as_tensor(params, dtype=torch.float32, device=dev).clone())
    pts = torch.as_tensor(points, dtype=torch.float32, device=dev).contiguous()
    xy = torch.as_tensor(ic_xy, dtype=torch.float32, device=dev).contiguous()
    opt = torch.optim.Adam([p], lr=lr)
    sched = _scheduler(opt)
    log = TrainLog()
    for _ in range(epochs):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        opt.zero_grad(set_to_none=False)
        if total:
            r = circuit.total_loss(p.detach(), pts, xy, desc)
            p.grad = r["grad"].clone()
            terms = r["terms"]
        else:
            r = circuit.maxwell(p.detach(), pts, desc.phys, outputs=False)
            p.grad = r["grad"].clone()
            terms = r["loss"]
        opt.step()
        sched.step()
        torch.cuda.synchronize()
        log.seconds.append(time.perf_counter() - t0)
        t = terms.cpu().tolist()
        log.loss.append(t[0])
        log.terms.append(tuple(t[1:]) if total else (t[0], 0.0, 0.0, 0.0))
    return log


def hybrid_total_loss(model: HybridQPINN, points: torch.Tensor, ic_xy: torch.Tensor, desc) -> dict:
    """The four terms of eq. 2D_lossTot for the hybrid model (torch): residuals and energy from the
    fields and their derivatives at the collocation points, symmetry from the fields at the mirror
    images (the x-mirror terms for the vacuum loss only), IC from the fields at (0, x, y)."""
    phys_kind = int(desc.phys.kind)
    fields, dfields = model(points)
    phys = maxwell_residual_loss(dfields, points, phys_kind, desc.phys.eps_r, desc.phys.x_interface)
    E, Hx, Hy = fields[:, :3].unbind(1)
    eps = torch.ones_like(E)
    if phys_kind:
        eps = torch.where(points[:, 1] >= desc.phys.x_interface, torch.full_like(E, desc.phys.eps_r), eps)
    Et, Ex, Ey, Hxt, _, Hxy, Hyt, Hyx, _ = dfields[:, :3, :3].flatten(1).unbind(1)
    e = (eps * E * Et + Hx * Hxt + Hy * Hyt) - (Ex * Hy + E * Hyx) + (Ey * Hx + E * Hxy)
    energy = torch.mean(e ** 2)
    my = points.clone()
    my[:, 2] = -my[:, 2]
    at = [my]
    if phys_kind == 0:
        mx = points.clone()
        mx[:, 1] = -mx[:, 1]
        at.append(mx)
    at.append(torch.cat([torch.zeros_like(ic_xy[:, :1]), ic_xy], dim=1))
    # the fields away from the collocation points in one evaluation, where the model is a map point by point
    plain = getattr(model, "plain_model", None)
    if plain is not None and plain():
        f = torch.split(model.fields(torch.cat(at)), [len(p) for p in at])
    else:
        f = [model.fields(p) for p in at]
    E1, Hx1, Hy1 = f[0][:, :3].unbind(1)
    sym = (E - E1) ** 2 + (Hx + Hx1) ** 2 + (Hy - Hy1) ** 2
    if phys_kind == 0:
        E2, Hx2, Hy2 = f[1][:, :3].unbind(1)
        sym = sym + (E - E2) ** 2 + (Hx - Hx2) ** 2 + (Hy + Hy2) ** 2
    sym = torch.mean(sym)
    Ei, Hxi, Hyi = f[-1][:, :3].unbind(1)
    E0 = torch.exp(-desc.ic_a * (ic_xy[:, 0] ** 2 + ic_xy[:, 1] ** 2))
    ic = torch.mean((Ei - E0) ** 2 + Hxi ** 2 + Hyi ** 2)
    total = phys + desc.w_ic * ic + desc.w_sym * sym + desc.w_energy * energy
    return {"total": total, "phys": phys, "ic": ic, "sym": sym, "energy": energy}


def train_hybrid(model: HybridQPINN, points, ic_xy, desc, epochs: int, lr: float = 1e-3) -> TrainLog:
    """Adam over every parameter of the hybrid model (network, circuit, head) on the full batch."""
    dev = next(model.parameters()).device
    pts = torch.as_tensor(points, dtype=torch.float32, device=dev).contiguous()
    xy = torch.as_tensor(ic_xy, dtype=torch.float32, device=dev).contiguous()
    opt = torch.optim.Adam(model.parameters(), lr=lr)
    sched = _scheduler(opt)
    log = TrainLog()
    for _ in range(epochs):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        opt.zero_grad(set_to_none=True)
        terms = hybrid_total_loss(model, pts, xy, desc)
        terms["total"].backward()
        opt.step()
        sched.step()
        torch.cuda.synchronize()
        log.seconds.append(time.perf_counter() - t0)
        log.loss.append(float(terms["total"].detach()))
        log.terms.append(tuple(float(terms[k].detach()) for k in ("phys", "ic", "sym", "energy")))
    return log


def grid_points(side: int, t_range=(0.0, 1.5), device=None) -> torch.Tensor:
    """The paper's equally spaced side^3 collocation grid: t in t_range, x and y over the periodic
    domain [-1, 1) (section "Maxwell's equations in two dimensions and problem setup")."""
    t = torch.linspace(t_range[0], t_range[1], side)
    s = -1.0 + 2.0 * torch.arange(side) / side
    T, X, Y = torch.meshgrid(t, s, s, indexing="ij")
    return torch.stack([T.ravel(), X.ravel(), Y.ravel()], 1).to(device)


def ic_plane(side: int, device=None) -> torch.Tensor:
    s = -1.0 + 2.0 * torch.arange(side) / side
    X, Y = torch.meshgrid(s, s, indexing="ij")
    return torch.stack([X.ravel(), Y.ravel()], 1).to(device)


def black_hole_indicator(U: torch.Tensor, t: torch.Tensor, delta: float) -> float:
    """I_BH = 1 - min_{t >= delta} U(t) / U(0) (t must contain 0)."""
    U = U.double().cpu()
    t = t.double().cpu()
    i0 = int(torch.argmin(t.abs()))
    if float(t[i0]) != 0.0:
        raise ValueError("the time slices must include t = 0")
    sel = t >= delta
    return float(1.0 - torch.min(U[sel] / U[i0]))


def hybrid_energy_profile(model: HybridQPINN, t: torch.Tensor, xg: torch.Tensor, yg: torch.Tensor,
                          eps_r: float = 1.0, x_interface: float = 0.0, dielectric: bool = False) -> torch.Tensor:
    """U(t) of the hybrid model's fields over the grid (float64 sums)."""
    dev = next(model.parameters()).device
    T, X, Y = torch.meshgrid(t, xg, yg, indexing="ij")
    pts = torch.stack([T.ravel(), X.ravel(), Y.ravel()], 1).to(dev)
    with torch.no_grad():
        f = model.fields(pts).double()
    eps = torch.ones_like(f[:, 0])
    if dielectric:
        eps = torch.where(pts[:, 1] >= x_interface, torch.full_like(eps, eps_r), eps)
    u = 0.5 * (eps * f[:, 0] ** 2 + f[:, 1] ** 2 + f[:, 2] ** 2)
    return u.reshape(len(t), -1).sum(1)
