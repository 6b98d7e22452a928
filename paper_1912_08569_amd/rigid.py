"""Rigid planar bodies on a System (the patchy colloids of Sec. 3.2).

A body is a disk (its centre particle) with massless member particles at fixed
body-frame offsets; both are particles of the System.  Each step launches the
stand-alone force kernel on every particle and the body kernel for the two BAOAB
halves (``rc_rigid_run``); the list is rebuilt when a path length passes the soft
skin threshold.  Every step runs in the library's HIP kernels; this module only
holds the body arrays and builds the lists in between.
"""
from __future__ import annotations

import operator
import time

import numpy as np
import torch

from . import _lib as rcl
from . import api


#: steps of one library call at most: its count is a C int, and a signal is seen between calls only
_CALL_STEPS = 1 << 20


class RigidBodies:
    def __init__(self, system, bodies: dict, theta, omega):
        """bodies: centre [B], first [B+1], member [M], offset [M, 2], inertia [B] (tags; host arrays)."""
        dev = system.device
        self.S = system
        self.b = {k: torch.as_tensor(np.ascontiguousarray(bodies[k]), device=dev)
                  for k in ("centre", "first", "member", "offset", "inertia")}
        for k in ("centre", "first", "member"):
            self.b[k] = self.b[k].to(torch.int32)
        self.b["offset"] = self.b["offset"].to(torch.float32).contiguous()
        self.b["inertia"] = self.b["inertia"].to(torch.float32)
        self.theta = torch.as_tensor(np.asarray(theta, np.float32), device=dev).clone()
        self.omega = torch.as_tensor(np.asarray(omega, np.float32), device=dev).clone()

    def run(self, n_steps: int, cfg, step0: int = 0, soft_frac: float = 0.8) -> dict:
        """n_steps body steps (cfg: an integrator of dim 2); returns rebuild count and wall time."""
        S = self.S
        n_steps = operator.index(n_steps)
        if not S.built:
            S.build()
        soft = 0.5 * S.r_buff * soft_frac
        S.compute_forces(gather=True, ev=False)
        rebuilds = 0
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        k, pending = 0, False
        while k < n_steps:
            steps = min(n_steps - k, _CALL_STEPS)
            code, done = api.rc_rigid_run(S.ctx, S.pos, S.vel, S.force, S.image, S.rtag, S.nlist, S.nn, self.b,
                                          self.theta, self.omega, S.box, cfg, step0 + k, steps, pending, soft,
                                          S.status)
            k += done
            pending = done < steps
            if code != rcl.RC_OK:
                raise RuntimeError(f"rigid bodies: non-finite state at step {step0 + k}")
            if pending:          # step k has its first half and waits for a list
                S.build()
                rebuilds += 1
        torch.cuda.synchronize()
        return {"rebuilds": rebuilds, "seconds": time.perf_counter() - t0}
