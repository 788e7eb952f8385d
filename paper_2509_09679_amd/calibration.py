"""One calibration step of the learnable butterfly rotation on a single linear layer, built from the
library's calls (paper, sections "Loss Function", "Uniformity Regularization" and "Implementation Details").

    L_recon   = || X W^T - Dequant(Quant(B X)) . Dequant(Quant(W B^T))^T ||^2      (rows of X are tokens)
    L_uniform = D_KL(P_bins || U): P_bins the occupancy of the 2^b activation code bins, U uniform

L_uniform is evaluated from the histogram the fake-quantising kernel counts in the same pass and is REPORTED beside
L_recon; it is not differentiated (the paper does not say how a gradient passes the hard bin assignment), so the
descent direction is that of L_recon alone.

16-bit rows: the dense products take the 16-bit matrices as they are and accumulate in float32; the float32 error matrix
enters its two products as a sum of 16-bit pieces (bq_residual_split).  As float32 products the four were 14.7 of the 16.8 ms
of a step (16384 rows, n = m = 4096, binary16).

The butterfly work — B X, W B^T (the forward transform over the rows of W), both fake quantisations and both
backward passes — runs in the HIP library; torch supplies memory, the two dense products with W (they
belong to the layer, not to the transform) and the element-wise rule that carries the loss gradient from
the fake-quantised values back to the rotated values.

The paper does not say how gradients pass `round` and the scale.  Reading taken here (what automatic
differentiation of  s * round(v / s),  s = max|v| / qmax,  gives with a straight-through `round`): with
g = dL/d(Dequant(Quant(v))) on a group,
    dL/dv_j = g_j                                          (straight-through),
    dL/dv_m += sign(v_m) / qmax * sum_j g_j (q_j - v_j / s)   for m = argmax |v|   (through the scale),
the binary16 rounding of s being treated as the identity.  Without the second term the gradient cannot see
that a rotation which lowers the group maxima lowers the quantisation noise: (W B^T)(B x) = W x for every
theta, so the straight-through term alone only sees noise cross terms.  SGD with a cosine learning-rate
schedule from theta = 0 (identity), as in the paper's set-up.
"""
from __future__ import annotations

import math
from dataclasses import dataclass

from . import binding as B


@dataclass
class QuantSpec:
    bits: int
    group: int
    scale_dtype: str = "f16"


class ButterflyCalibrator:
    """Holds theta (float32, [1][k][n/2]) for one layer and the buffers of a step.  X: [T, n], W: [m, n], both
    of the same 16-bit or 32-bit row type, resident on the GPU."""

    def __init__(self, W, act: QuantSpec, wgt: QuantSpec, theta=None):
        import torch

        self.torch = torch
        self.W = W
        self.m, self.n = W.shape
        self.k = self.n.bit_length() - 1
        assert 1 << self.k == self.n
        self.act, self.wgt = act, wgt
        dev = W.device
        self.theta = (torch.zeros((1, self.k, self.n // 2), dtype=torch.float32, device=dev)
                      if theta is None else theta.clone())
        self.plan = torch.empty(B.bq_plan_bytes(self.n, 1), dtype=torch.uint8, device=dev)
        self.Wq = torch.empty_like(W)
        self.dW = torch.empty_like(W)
        self.dth_x = torch.empty_like(self.theta)
        self.dth_w = torch.empty_like(self.theta)
        self.hist = torch.zeros(1 << act.bits, dtype=torch.int64, device=dev)
        self._ws = None

    def _workspace(self, rows):
        need = max(256, B.bq_butterfly_bwd_workspace_bytes(rows))
        if self._ws is None or self._ws.numel() < need:
            self._ws = self.torch.empty(need, dtype=self.torch.uint8, device=self.W.device)
        return self._ws

    def _half_step(self, X, Xq, V, Wr):
        """The step between the fake quantisations and the backward passes for 16-bit rows: (L_recon, dL/dV, dL/dWr), the
        gradients in float32."""
        torch = self.torch
        T, m, dev = X.shape[0], self.m, X.device
        f32 = torch.float32
        E = torch.mm(X, self.W.t(), out_dtype=f32)
        E = torch.addmm(E, Xq, self.Wq.t(), beta=-1.0, out_dtype=f32, out=E)
        ld = (m + 7) // 8 * 8
        P = torch.empty((2 if X.dtype == torch.float16 else 3, T, ld), dtype=X.dtype, device=dev)
        res = torch.empty(2, dtype=f32, device=dev)
        scratch = torch.empty(B.bq_residual_scratch_bytes(), dtype=torch.uint8, device=dev)
        step = B.RESIDUAL_STEP["f16" if X.dtype == torch.float16 else "bf16"]
        B.bq_residual_split(E, P, res, scratch)
        del E
        grads = []
        for A, Q, R, spec, transposed in ((self.Wq, Xq, V, self.act, False), (Xq, self.Wq, Wr, self.wgt, True)):
            G = None
            for piece in reversed(P[:, :, :m].unbind(0)):  # the smallest piece first
                piece = piece.t() if transposed else piece
                G = torch.mm(piece, A, out_dtype=f32) if G is None else torch.addmm(G, piece, A, beta=step, out_dtype=f32,
                                                                                     out=G)
            if 8 <= spec.group <= 8192:
                B.bq_quantiser_grad(R, Q, G, res[1:], B.make_quant(spec.bits, spec.group, spec.scale_dtype),
                                    B.make_rows(R, self.n, 1))
            else:
                G = self._through_quantiser(R.float(), Q.float(), G * res[1], spec)
            grads.append(G)
        return res[0], grads[0], grads[1]

    def _through_quantiser(self, V, Vq, G, spec: QuantSpec):
        """dL/dV from G = dL/dVq (all float32, [rows, n]); see the module text."""
        torch = self.torch
        rows, n = V.shape
        g = spec.group
        qmax = float((1 << (spec.bits - 1)) - 1)
        v = V.reshape(rows, n // g, g)
        amax, idx = v.abs().max(dim=-1, keepdim=True)
        s = amax / qmax
        ok = s > 0
        inv = torch.where(ok, 1.0 / torch.where(ok, s, torch.ones_like(s)), torch.zeros_like(s))
        r = (Vq.reshape(rows, n // g, g) - v) * inv  # q_j - v_j / s
        Gg = G.reshape(rows, n // g, g)
        through_scale = (Gg * r).sum(dim=-1, keepdim=True) * torch.sign(torch.gather(v, -1, idx)) / qmax
        dV = Gg.clone()
        dV.scatter_add_(-1, idx, through_scale)
        return dV.reshape(rows, n)

    def _bwd_f32(self, X, dV, dtheta):
        """dtheta from (X, dL/dV) with float32 rows: the gradient's entries span many orders of magnitude (the
        term through the scale sits on one element per group), which a 16-bit row type would flush to zero."""
        X32 = X.float().contiguous()  # rows as far apart as dV's
        rows = B.make_rows(X32, self.n, 1)
        B.bq_butterfly_bwd(X32, dV.contiguous(), self.plan, None, dtheta, self._workspace(rows), rows)
        return dtheta

    def uniformity_kl(self):
        """D_KL(P_bins || U) of the activation codes of the last loss_and_grad call, from the kernel's histogram
        (0 log 0 = 0); a 0-dim float64 tensor."""
        torch = self.torch
        h = self.hist.to(torch.float64)
        p = h / h.sum().clamp_min(1.0)
        bins = float(1 << self.act.bits)
        return torch.where(p > 0, p * torch.log(p.clamp_min(1e-300) * bins), torch.zeros_like(p)).sum()

    def loss_and_grad(self, X):
        """Returns (L_recon as a 0-dim float32 tensor, dtheta of L_recon, L_uniform as a 0-dim float64 tensor);
        self.hist holds the activation code bins."""
        torch = self.torch
        B.bq_plan_build(self.theta, self.n, 1, self.plan)
        V, Xq, Wr = torch.empty_like(X), torch.empty_like(X), torch.empty_like(self.W)  # dense also where X or W is not
        rx, rw = B.make_rows(X, self.n, 1, out=V), B.make_rows(self.W, self.n, 1, out=Wr)
        qa = B.make_quant(self.act.bits, self.act.group, self.act.scale_dtype)
        qw = B.make_quant(self.wgt.bits, self.wgt.group, self.wgt.scale_dtype)
        B.bq_butterfly_fwd(X, V, self.plan, rx)
        B.bq_butterfly_fwd_fakequant(X, self.plan, Xq, self.hist, qa, rx)
        B.bq_butterfly_fwd(self.W, Wr, self.plan, rw)
        B.bq_butterfly_fwd_fakequant(self.W, self.plan, self.Wq, None, qw, rw)
        # the layer's dense products (float32 accumulate)
        # autograd through the loss, reverse or forward: the 16-bit products have no derivative
        tangent = torch.autograd.forward_ad.unpack_dual
        tracked = (torch.is_grad_enabled() and (X.requires_grad or self.W.requires_grad)) or any(
            tangent(t).tangent is not None for t in (X, self.W))
        # the float32 products work on copies; the 16-bit ones on X and W as they lie, which are left to them only 16-byte aligned
        aligned = all(t.data_ptr() % 16 == 0 and t.stride(0) % 8 == 0 for t in (X, self.W))
        if X.dtype != torch.float32 and X.dtype == self.W.dtype and X.shape[0] > 0 and self.m > 0 and aligned and not tracked:
            loss, dV, dWr = self._half_step(X, Xq, V, Wr)
        else:
            Xq32, Wq32 = Xq.float(), self.Wq.float()
            E = (Xq32 @ Wq32.t()) - (X.float() @ self.W.float().t())
            loss = (E * E).sum()
            dV = self._through_quantiser(V.float(), Xq32, 2.0 * (E @ Wq32), self.act)
            dWr = self._through_quantiser(Wr.float(), Wq32, 2.0 * (E.t() @ Xq32), self.wgt)
        gx = self._bwd_f32(X, dV, self.dth_x)
        gw = self._bwd_f32(self.W, dWr, self.dth_w)
        self.Xq = Xq
        return loss, gx + gw, self.uniformity_kl()

    def fit(self, X, steps: int, lr: float, log=None):
        """SGD with a cosine learning-rate schedule; returns the losses seen (before each update).  The step
        is lr times the unit-norm gradient (this module's choice: the loss scale varies by orders of
        magnitude with the batch and layer size, the paper gives no learning rate)."""
        losses = []
        self.kl_seen = []
        for t in range(steps):
            loss, g, kl = self.loss_and_grad(X)
            losses.append(float(loss))
            self.kl_seen.append(float(kl))
            step_lr = 0.5 * lr * (1.0 + math.cos(math.pi * t / steps))
            gn = g.norm()
            self.theta -= step_lr * g / (gn + 1e-30)
            if log:
                log(t, losses[-1])
        return losses
