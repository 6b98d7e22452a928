"""torch.autograd bindings: energy, forces and the soft bond count as
differentiable functions of the positions and of the per-entry parameters.

Positions are (N, 3) float32 device tensors in tag order (the engine's own
order changes at every list build; ``SwapModel`` maps between the two).  The
parameters are an (nt, nt, 3) float64 CPU tensor theta = (eps, sigma, lambda)
per entry; entry {a, b} is read from theta[min(a,b), max(a,b)] and its
gradient is reported there (the lower triangle gets zeros).  Every value and
derivative comes from the HIP library:

  energy   E(x, theta):  dE/dx = -F,  dE/dtheta = rc_param_grad
  forces   F(x, theta):  a . dF/dx = -H a (rc_force_hvp),  a . dF/dtheta = rc_param_vjp
  soft bonds B(x):        dB/dx = rc_soft_bonds' gradient
"""
from __future__ import annotations

import numpy as np
import torch

from . import _lib as rcl
from . import api


class SwapModel:
    """A ``System`` seen through tag-ordered positions and a parameter tensor.

    Keeps the neighbour list valid: a call whose positions moved more than
    half the skin (minimum image) from those of the last build rebuilds it.
    """

    def __init__(self, system):
        self.S = system
        self.L = torch.tensor(system.edges, dtype=torch.float32, device=system.device)
        self.half_skin = 0.5 * system.ctx.r_buff
        self.base = system.table.copy()
        self._theta = None
        system.build()
        self._ref = self._to_tag(system.pos)    # positions of the last build, by tag
        self.rebuilds = 0

    def positions(self) -> torch.Tensor:
        """Current positions of the system in tag order (N, 3)."""
        return self._to_tag(self.S.pos)

    # ---- parameters ---------------------------------------------------------------------------
    def theta(self) -> torch.Tensor:
        t = self.base
        return torch.tensor(np.stack([t.epsilon, t.sigma, t.lam], axis=-1), dtype=torch.float64)

    def _load_theta(self, theta: torch.Tensor):
        th = theta.detach().cpu().numpy().astype(np.float64)
        if self._theta is not None and np.array_equal(th, self._theta):
            return
        nt = th.shape[0]
        tab = self.base.copy()
        for a in range(nt):
            for b in range(nt):
                lo, hi = min(a, b), max(a, b)
                if tab.kind[a, b] == 0:
                    continue
                tab.epsilon[a, b], tab.sigma[a, b] = th[lo, hi, 0], th[lo, hi, 1]
                tab.lam[a, b] = th[lo, hi, 2] if tab.kind[a, b] == rcl.RC_KIND_SWAP else tab.lam[a, b]
        self.S.set_table(tab)
        self._theta = th

    @staticmethod
    def _upper(g: np.ndarray) -> torch.Tensor:
        nt = g.shape[0]
        out = np.zeros_like(g)
        iu = np.triu_indices(nt)
        out[iu] = g[iu]
        return torch.from_numpy(out)

    # ---- positions ----------------------------------------------------------------------------------
    def _by_tag(self, t: torch.Tensor) -> torch.Tensor:
        """t as a contiguous (N, 3) float32 tensor."""
        if t.dim() != 2 or t.shape[0] != self.S.N:
            raise RuntimeError(f"expected ({self.S.N}, 3) values by tag, not {tuple(t.shape)}")
        return t.detach().to(torch.float32).expand(self.S.N, 3).contiguous()

    def _on_list(self, xyz: torch.Tensor, evaluate):
        """evaluate() on the positions xyz with a list valid for them.

        It is queued behind the load at once, so that the host's wait for the moved flag is over by the
        time it is done; positions that had moved too far get a list and are evaluated again."""
        S = self.S
        S.invalidate()   # positions written here, outside the driver
        api.rc_load_by_tag(S.ctx, S.pos, self._by_tag(xyz), self._ref, S.box, self.half_skin)
        out = evaluate()
        if api.rc_load_moved(S.ctx):
            S.build()
            self._ref = self._to_tag(S.pos)
            self.rebuilds += 1
            out = evaluate()
        return out

    def _to_tag(self, arr, negate=False):
        return api.rc_to_tags(self.S.ctx, arr, self.S.rtag, negate)

    def _to_engine(self, a_tag):
        return api.rc_from_tags(self.S.ctx, self._by_tag(a_tag), self.S.pos)

    # ---- evaluations (tag order) ---------------------------------------------------------------
    def load(self, xyz, theta):
        """The state that hvp, param_grad and param_vjp are taken at."""
        self._load_theta(theta)
        self._on_list(xyz, lambda: None)

    def forces_energy(self, xyz, theta, negate=False):
        """(forces, energy), or (minus the forces, energy)."""
        def evaluate():
            F, ev = self.S.compute_forces(gather=True)
            return self._to_tag(F, negate), ev[0].clone()
        self._load_theta(theta)
        return self._on_list(xyz, evaluate)

    def hvp(self, v_tag):
        return self._to_tag(self.S.hvp(self._to_engine(v_tag)))

    def param_grad(self):
        return self._upper(self.S.param_grad())

    def param_vjp(self, a_tag):
        return self._upper(self.S.param_vjp(self._to_engine(a_tag)))

    def energy_theta_grad(self, xyz, theta, gE):
        """gE dE/dtheta."""
        self._load_theta(theta)
        g = self._on_list(xyz, lambda: self.S.param_grad_tensor() * gE.detach())
        return self._upper(g.cpu().numpy())

    def forces_grads(self, xyz, theta, gF, want_x, want_theta):
        """gF . dF/dx and gF . dF/dtheta (None where not wanted)."""
        def evaluate():
            a = self._to_engine(gF)
            gx = self._to_tag(self.S.hvp(a), negate=True) if want_x else None
            return gx, self.S.param_vjp_tensor(a) if want_theta else None
        self._load_theta(theta)
        gx, gt = self._on_list(xyz, evaluate)
        return gx, self._upper(gt.cpu().numpy()) if want_theta else None

    def soft_bonds(self, xyz):
        def evaluate():
            val, g = self.S.soft_bonds(grad=True)
            return val[0], self._to_tag(g)
        val, g = self._on_list(xyz, evaluate)
        return val.clone(), g


class _Energy(torch.autograd.Function):
    @staticmethod
    def forward(ctx, xyz, theta, model):
        G, E = model.forces_energy(xyz, theta, negate=True)     # the gradient is minus the forces
        ctx.model = model
        ctx.save_for_backward(xyz, theta, G)
        return E

    @staticmethod
    def backward(ctx, gE):
        xyz, theta, G = ctx.saved_tensors
        gx = gt = None
        if ctx.needs_input_grad[0]:
            gx = G * gE.to(G.dtype)
        if ctx.needs_input_grad[1]:
            gt = ctx.model.energy_theta_grad(xyz, theta, gE)
        return gx, gt, None


class _Forces(torch.autograd.Function):
    @staticmethod
    def forward(ctx, xyz, theta, model):
        F, _ = model.forces_energy(xyz, theta)
        ctx.model = model
        ctx.save_for_backward(xyz, theta)
        return F

    @staticmethod
    def backward(ctx, gF):
        xyz, theta = ctx.saved_tensors
        gx, gt = ctx.model.forces_grads(xyz, theta, gF, ctx.needs_input_grad[0], ctx.needs_input_grad[1])
        return gx, gt, None


class _SoftBonds(torch.autograd.Function):
    @staticmethod
    def forward(ctx, xyz, model):
        B, g = model.soft_bonds(xyz)
        ctx.save_for_backward(g)
        return B

    @staticmethod
    def backward(ctx, gB):
        (g,) = ctx.saved_tensors
        return g * gB.to(g.dtype), None


def swap_energy(model: SwapModel, xyz: torch.Tensor, theta: torch.Tensor) -> torch.Tensor:
    """Total energy (float64 scalar), differentiable in xyz and theta."""
    return _Energy.apply(xyz, theta, model)


def swap_forces(model: SwapModel, xyz: torch.Tensor, theta: torch.Tensor) -> torch.Tensor:
    """Forces (N, 3) float32 in tag order, differentiable in xyz and theta."""
    return _Forces.apply(xyz, theta, model)


def soft_bonds(model: SwapModel, xyz: torch.Tensor) -> torch.Tensor:
    """Soft bond count (float64 scalar), differentiable in xyz."""
    return _SoftBonds.apply(xyz, model)
