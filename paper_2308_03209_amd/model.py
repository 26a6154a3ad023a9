"""Buffers and call sequence of one training iteration on one partition (Algorithm 1 lines 6-12).

This module only allocates device memory with torch and issues the library's calls in
order: layer_fwd x L, loss_weighted, layer_bwd x L, step.  All arithmetic runs in the HIP
kernels behind `binding`.
"""
from __future__ import annotations

from typing import Dict, List, Optional, Sequence, Tuple

import numpy as np
import torch

from . import binding as B

_KIND = {"gcn": B.GCN, "sage": B.SAGE_MEAN, "sage_conv": B.SAGE_CONV}
_DTYPE = {"f32": (B.F32, torch.float32), "bf16": (B.BF16, torch.bfloat16)}
_NAMES = {"gcn": ("W", "bW"), "sage": ("W", "bW", "U", "bU"), "sage_conv": ("W", "bW")}


def param_shapes(kind: str, dims: Sequence[Tuple[int, int, int]]) -> List[Dict[str, Tuple[int, ...]]]:
    out = []
    for (d_in, d_msg, d_out) in dims:
        if kind == "sage":
            out.append({"W": (d_msg, d_in), "bW": (d_msg,), "U": (d_out, d_msg + d_in), "bU": (d_out,)})
        elif kind == "sage_conv":
            out.append({"W": (d_out, 2 * d_in), "bW": (d_out,)})
        else:
            out.append({"W": (d_out, d_in), "bW": (d_out,)})
    return out


class Model:
    """Parameters, gradients and Adam state as single flat float32 device buffers with per-tensor views."""

    def __init__(self, kind: str, dims: Sequence[Tuple[int, int, int]], device="cuda"):
        self.kind = kind
        self.dims = list(dims)
        self.shapes = param_shapes(kind, dims)
        total = 0
        self.slices = []
        for layer in self.shapes:
            sl = {}
            for name in _NAMES[kind]:
                n = int(np.prod(layer[name]))
                n_pad = (n + 63) // 64 * 64          # keep every tensor 256-byte aligned
                sl[name] = (total, n, layer[name])
                total += n_pad
                self.total = sl[name][0] + n         # elements that a flat buffer has to have
            self.slices.append(sl)
        self.theta = torch.zeros(total, dtype=torch.float32, device=device)
        self.grad = torch.zeros(total, dtype=torch.float32, device=device)
        # byte offset of every tensor in the flat buffers, per layer (W, bW, U, bU; None where the kind has none)
        self.offsets = [tuple(4 * sl[k][0] if k in sl else None for k in ("W", "bW", "U", "bU")) for sl in self.slices]
        self.m = None
        self.v = None
        self.t = 0

    def _views(self, flat) -> List[Dict[str, torch.Tensor]]:
        return [{k: flat[o:o + n].view(shape) for k, (o, n, shape) in sl.items()} for sl in self.slices]

    def flat_ptr(self, flat: torch.Tensor) -> int:
        """Address of `theta` or `grad`, which a program may have put in its place: it has to hold every tensor."""
        if flat.numel() < self.total:
            raise ValueError(f"flat buffer of {flat.numel()} elements for {self.total}")
        return B._ptr(flat)

    @property
    def params(self):
        return self._views(self.theta)

    @property
    def grads(self):
        return self._views(self.grad)

    def load(self, layers: Sequence[Dict[str, np.ndarray]]) -> None:
        for views, src in zip(self.params, layers):
            for k, v in views.items():
                v.copy_(torch.from_numpy(np.ascontiguousarray(src[k], dtype=np.float32)))

    def step(self, kind: int = B.SGD, lr: float = 0.01, b1=0.9, b2=0.999, eps=1e-8) -> None:
        if kind == B.ADAM and self.m is None:
            self.m = torch.zeros_like(self.theta)
            self.v = torch.zeros_like(self.theta)
        self.t += 1
        B.step(kind, self.theta, self.grad, self.m, self.v, lr, b1, b2, eps, self.t)


class BufferPool:
    """Device buffers shared by the runners of several partitions that are trained one after the other:
    every request is served from one allocation per (tag, columns, dtype), sized for the largest partition."""

    def __init__(self, max_rows: int, device="cuda"):
        self.max_rows, self.device, self.bufs = int(max_rows), device, {}

    def rows(self, tag, n: int, cols: int, dtype) -> torch.Tensor:
        key = (tag, cols, dtype)
        if key not in self.bufs:
            self.bufs[key] = torch.empty((self.max_rows, cols), dtype=dtype, device=self.device)
        return self.bufs[key][:n]

    def raw(self, tag, nbytes: int) -> torch.Tensor:
        key = (tag, "raw")
        if key not in self.bufs or self.bufs[key].numel() < nbytes:
            self.bufs[key] = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
        return self.bufs[key]


class PartitionRunner:
    """Activation / scratch buffers of one partition and the forward-loss-backward call sequence."""

    def __init__(self, part: B.Partition, model: Model, masks: Optional[B.Masks] = None, dropout_q: float = 0.0,
                 dropout_seed: int = 0, device="cuda", dtype: str = "f32", pool: Optional[BufferPool] = None,
                 loss: str = "softmax_ce", fuse_gates: bool = True):
        """loss: "softmax_ce" (labels int32 [n]) or "sigmoid_bce" (multi-label targets uint8 [n, C]).
        fuse_gates: between two layers that end in ReLU, the upper layer's backward writes its input
        gradient already gated and scaled by the lower layer's ReLU and dropout (one elementwise pass
        less per layer).
        dtype: storage of features / activations / activation gradients ("f32" or "bf16");
        parameters, their gradients and the loss are always float32.  pool: share buffers with the runners
        of other partitions (which then must not run concurrently)."""
        self.part, self.model, self.masks = part, model, masks
        if loss not in ("softmax_ce", "sigmoid_bce"):
            raise ValueError(loss)
        self.loss_kind = loss
        self.fuse_gates = bool(fuse_gates)
        self.q, self.dseed = float(dropout_q), int(dropout_seed)
        self.dtype_code, self.torch_dtype = _DTYPE[dtype]
        n = part.num_nodes
        self.n = n
        L = len(model.dims)
        td = self.torch_dtype

        def buf(tag, cols):
            if pool is not None:
                return pool.rows(tag, n, cols, td)
            return torch.empty((n, cols), dtype=td, device=device)

        self.H = [None] + [buf(("H", l), d_out) for l, (_, _, d_out) in enumerate(model.dims)]
        self.saved = []
        for l, (d_in, d_msg, d_out) in enumerate(model.dims):
            if model.kind == "sage":
                self.saved.append({"Z": buf(("Z", l), d_msg), "A": buf(("A", l), d_msg)})
            elif d_in <= d_out:
                self.saved.append({"A": buf(("A", l), d_in)})
            else:
                self.saved.append({})
        # gradient w.r.t. each layer's input (none for the first layer: features need no gradient);
        # a layer's input gradient is dead once the layer below has consumed it, so two buffers alternate
        self.dH = [None] + [buf(("dH", l % 2), d_in) for l, (d_in, _, _) in enumerate(model.dims[1:], start=1)]
        self.dlogits = buf(("dlogits", 0), model.dims[-1][2])
        self._calls = (B.LayerCall * L)()
        self._calls_for = None   # settings the descriptors in _calls were made from
        self.loss = torch.zeros(1, dtype=torch.float32, device=device)
        ws = max(B.loss_workspace_bytes(), B.layers_workspace_bytes([self.desc(l, 0) for l in range(L)], n))
        self.workspace = pool.raw("workspace", ws) if pool is not None else torch.empty(ws, dtype=torch.uint8,
                                                                                        device=device)

    def desc(self, l: int, epoch: int) -> B.LayerDesc:
        d_in, d_msg, d_out = self.model.dims[l]
        last = l == len(self.model.dims) - 1
        act = 1 if (self.model.kind in ("gcn", "sage_conv") and not last) else 0
        q = 0.0 if last else self.q
        flags, q_below = 0, 0.0
        if self.fuse_gates and self.model.kind in ("gcn", "sage_conv"):
            if l > 0:
                flags |= B.GRAD_IN_GATED    # layer l-1 ends in ReLU and dropout with rate self.q
                q_below = self.q
            if not last:
                flags |= B.GRAD_OUT_GATED   # layer l+1 gates and scales what it hands down
        return B.layer_desc(_KIND[self.model.kind], d_in, d_msg, d_out, act, q, l, self.dseed, epoch, self.dtype_code,
                            flags, q_below)

    def _layer_calls(self):
        settings = (self.q, self.dseed, self.fuse_gates, self.dtype_code)
        if settings != self._calls_for:
            for l, c in enumerate(self._calls):
                c.desc = self.desc(l, 0)
            self._calls_for = settings
        return self._calls

    def _fill(self, c: B.LayerCall, l: int, epoch: int, theta: int) -> None:
        """Addresses of layer l's buffers and parameters, taken anew for every call."""
        c.desc.epoch = epoch
        c.H_in, c.H_out = B._ptr(self.H[l]), B._ptr(self.H[l + 1])
        saved = self.saved[l]
        if "Z" in saved:
            c.saved.Z = B._ptr(saved["Z"])
        if "A" in saved:
            c.saved.A = B._ptr(saved["A"])
        W, bW, U, bU = self.model.offsets[l]
        p = c.params
        p.W, p.bW = theta + W, theta + bW
        if U is not None:
            p.U, p.bU = theta + U, theta + bU

    def forward(self, X: torch.Tensor, mask_id: int = 0, epoch: int = 0) -> torch.Tensor:
        if X.dtype != self.torch_dtype:
            raise ValueError(f"features must be {self.torch_dtype}")
        self.H[0] = X
        calls, theta = self._layer_calls(), self.model.flat_ptr(self.model.theta)
        for l, c in enumerate(calls):
            self._fill(c, l, epoch, theta)
        B.layers_fwd(self.part, self.masks, mask_id, calls, self.workspace)
        return self.H[-1]

    def loss_backward(self, labels: torch.Tensor, weight_kind: int = B.W_DAR, scale_c: float = 1.0,
                      mask_id: int = 0, epoch: int = 0, accumulate: bool = False, custom_w=None,
                      train_mask=None) -> None:
        C = self.model.dims[-1][2]
        loss_fn = B.loss_weighted if self.loss_kind == "softmax_ce" else B.loss_bce_weighted
        loss_fn(self.part, weight_kind, custom_w, self.H[-1], labels, train_mask, C, scale_c, self.loss,
                self.dlogits, self.workspace, self.dtype_code)
        theta, grad = self.model.flat_ptr(self.model.theta), self.model.flat_ptr(self.model.grad)
        d_out = B._ptr(self.dlogits)
        calls = self._layer_calls()
        for l in range(len(calls) - 1, -1, -1):
            c = calls[l]
            self._fill(c, l, epoch, theta)
            c.dH_out = d_out
            c.dH_in = d_out = B._ptr(self.dH[l])
            W, bW, U, bU = self.model.offsets[l]
            g = c.grads
            g.W, g.bW = grad + W, grad + bW
            if U is not None:
                g.U, g.bU = grad + U, grad + bU
        B.layers_bwd(self.part, self.masks, mask_id, calls, accumulate, self.workspace)

    def iteration(self, X, labels, epoch: int, mask_seed: int = 0, weight_kind: int = B.W_DAR,
                  scale_c: float = 1.0, accumulate: bool = False, custom_w=None) -> int:
        """Pick the iteration's mask, forward, loss, backward.  Returns the mask index used."""
        k = B.dropedge_pick(mask_seed, epoch, self.masks.count) if self.masks is not None else 0
        self.forward(X, k, epoch)
        self.loss_backward(labels, weight_kind, scale_c, k, epoch, accumulate, custom_w)
        return k
