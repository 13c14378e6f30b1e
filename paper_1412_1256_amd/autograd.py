"""Differentiation form: calibrated Stokes spectra as a torch.autograd.Function.

Forward: set the learnable window, integrate all frames of ``packed`` and form calibrated Stokes spectra
(Eq. 2 with gains and leakage).  Backward: ``ps_calibrate_backward``, which recomputes the per-frame
transforms instead of storing them.  Complex parameters are complex64 tensors; their gradients follow torch's
convention for real losses (dL/dRe + i dL/dIm).
"""
from __future__ import annotations

import torch

from . import Plan, PolarisError


class StokesFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, gain_x, gain_y, dterms, taps, plan: Plan, packed, psi: float):
        if taps is not None:
            plan.set_window_taps(taps.detach())
        plan.reset()
        # the calibration and the output are instance 0's; a plan's other instances only accumulate
        inst, others = plan.instances[0], [None] * (len(plan.instances) - 1)
        cal = tuple(None if t is None else t.detach() for t in (gain_x, gain_y, dterms)) + (psi,)
        iquv = torch.empty((inst.n_pairs, 4, inst.channels), dtype=torch.float32, device=plan.device)
        plan.accumulate_stokes(packed, outs=[iquv] + others, cals=[cal] + others)
        ctx.save_for_backward(*(t if t is not None else torch.empty(0) for t in (gain_x, gain_y, dterms, taps)))
        ctx.present = tuple(t is not None for t in (gain_x, gain_y, dterms, taps))
        ctx.plan, ctx.packed, ctx.psi = plan, packed, psi
        ctx.integration = plan.integration_id()
        return iquv

    @staticmethod
    def backward(ctx, g_iquv):
        if ctx.plan.integration_id() != ctx.integration:
            # another forward (or reset, accumulate, new taps) ran on the plan since this node's forward: its
            # accumulators and window are no longer this node's
            raise PolarisError(4, "the plan's integration changed after this forward; run the backward before "
                                  "the next forward on the same plan, or use one plan per forward")
        gx, gy, dt, taps = (t if p else None for t, p in zip(ctx.saved_tensors, ctx.present))
        plan = ctx.plan
        inst = plan.instances[0]
        d_gx = d_gy = d_dt = d_taps = None
        # complex gradients are written as the (re, im) pairs that complex64 tensors hold
        if ctx.needs_input_grad[0]:
            d_gx = torch.empty((inst.n_pairs, inst.channels), dtype=torch.complex64, device=plan.device)
        if ctx.needs_input_grad[1]:
            d_gy = torch.empty((inst.n_pairs, inst.channels), dtype=torch.complex64, device=plan.device)
        if ctx.needs_input_grad[2]:
            d_dt = torch.empty((inst.n_pairs, 2), dtype=torch.complex64, device=plan.device)
        if ctx.needs_input_grad[3] and inst.window == "taps":
            d_taps = torch.empty((inst.n_taps,), dtype=torch.float32, device=plan.device)
        plan._backward_into(dict(gain_x=d_gx, gain_y=d_gy, dterms=d_dt, taps=d_taps), ctx.packed, g_iquv, 0, gx, gy, dt,
                            ctx.psi)
        return d_gx, d_gy, d_dt, d_taps, None, None, None


def stokes(plan: Plan, packed, gain_x=None, gain_y=None, dterms=None, taps=None, psi: float = 0.0):
    """Differentiable calibrated Stokes spectra [P][4][C] of one integration of ``packed``."""
    return StokesFn.apply(gain_x, gain_y, dterms, taps, plan, packed, psi)
