"""Two-layer full-batch GCN whose sparse aggregations run through sd_spmm.

The paper's application study (Sec. "Evaluation", GCN paragraph) trains a
two-layer GCN on a normalised adjacency Â with four sparse aggregations per
epoch: Â·(X W1) and Â·(H1 W2) forward, Âᵀ·G at both widths backward. Only the
aggregation is replaced, and the weight gradients of the dense transforms (tall
products X^T dC, which the library's GEMM runs on a handful of workgroups);
everything else is ordinary torch operations.

Each aggregation is `spmm(B, fwd, bwd)`: C = Â·B with plan `fwd`, and in the
backward pass dB = Âᵀ·dC with the transpose plan `bwd` (A is not assumed
symmetric).  Plans are built once per (graph, width) and reused every epoch.
"""
from __future__ import annotations

import torch

from . import Plan, sd_gemm_tn, sd_gemm_tn_workspace, sd_plan_device, sd_plan_ex, sd_spmm


class _SpMM(torch.autograd.Function):
    @staticmethod
    def forward(ctx, B, fwd: Plan, bwd: Plan):
        info = fwd.info
        if B.dim() != 2 or B.shape[0] != info["k"] or B.shape[1] != info["n"] or B.dtype != torch.float32:
            raise ValueError(f"spmm: B must be float32 [{info['k']}, {info['n']}], got {tuple(B.shape)} {B.dtype}")
        B = B.contiguous()
        C = torch.empty((info["m"], info["n"]), dtype=torch.float32, device=B.device)
        sd_spmm(fwd, B, C, torch.cuda.current_stream(B.device))
        ctx.bwd = bwd
        return C

    @staticmethod
    def backward(ctx, dC):
        bwd = ctx.bwd
        info = bwd.info
        dC = dC.contiguous()
        dB = torch.empty((info["m"], info["n"]), dtype=torch.float32, device=dC.device)
        sd_spmm(bwd, dC, dB, torch.cuda.current_stream(dC.device))
        return dB, None, None


def spmm(B: torch.Tensor, fwd: Plan, bwd: Plan) -> torch.Tensor:
    """C = Â·B; its gradient with respect to B is Âᵀ·dC (plan `bwd`)."""
    return _SpMM.apply(B, fwd, bwd)


def _weight_grad(X: torch.Tensor, dC: torch.Tensor) -> torch.Tensor:
    """X^T dC by sd_gemm_tn."""
    X = X if X.stride(1) == 1 and X.stride(0) >= X.shape[1] else X.contiguous()
    dC = dC.contiguous()
    (rows, p), q = X.shape, dC.shape[1]
    dW = torch.empty((p, q), dtype=torch.float32, device=X.device)
    size = sd_gemm_tn_workspace(rows, p, q)
    work = torch.empty(size, dtype=torch.uint8, device=X.device)
    with torch.cuda.device(X.device):
        sd_gemm_tn(X, X.stride(0), dC, q, rows, p, q, dW, work, size, torch.cuda.current_stream(X.device))
    return dW


class _Transform(torch.autograd.Function):
    """X W, with its weight gradient by sd_gemm_tn.  A backward pass that is
    itself differentiated (create_graph) uses torch's products throughout."""

    @staticmethod
    def forward(ctx, X, W):
        ctx.save_for_backward(X, W)
        return X @ W

    @staticmethod
    def backward(ctx, dC):
        X, W = ctx.saved_tensors
        dX = dC @ W.t() if ctx.needs_input_grad[0] else None
        dW = None
        if ctx.needs_input_grad[1]:
            dW = X.t() @ dC if torch.is_grad_enabled() else _weight_grad(X, dC)
        return dX, dW


# Rows from which sd_gemm_tn beat torch's X^T dC at every width up to 256
# measured (128 x 128: 21 against 56 us at 10,000 rows, 116 against 487 at
# 262,144; 32 x 7: 22 against 36 and 61 against 350).  At 3,000 rows the two are
# within 4 us either way, and at width 602 within a tenth at a million rows.
_GRAD_ROWS, _GRAD_WIDTH = 8192, 256


def transform(X: torch.Tensor, W: torch.Tensor) -> torch.Tensor:
    """X @ W.  Many fp32 rows on the GPU take the native weight gradient; every
    other case (other types and devices, few rows, wide layers, autocast,
    function transforms, forward-mode or compiled tracing) is torch's own."""
    if (X.dim() == 2 and W.dim() == 2 and X.is_cuda and W.is_cuda and X.device == W.device
            and X.dtype == W.dtype == torch.float32 and type(X) in (torch.Tensor, torch.nn.Parameter)
            and X.layout == W.layout == torch.strided and W.requires_grad and torch.is_grad_enabled()
            and X.shape[1] == W.shape[0] and X.shape[0] >= _GRAD_ROWS
            and 1 <= W.shape[0] <= _GRAD_WIDTH and 1 <= W.shape[1] <= _GRAD_WIDTH
            and not torch.is_autocast_enabled() and not torch.compiler.is_compiling()
            and not torch._C._are_functorch_transforms_active()
            and torch.autograd.forward_ad._current_level < 0):
        return _Transform.apply(X, W)
    return X @ W


class AggregationPlans:
    """Forward and transpose plans of one adjacency for each width used.

    A is a host CSR (an object with m, k, rowptr, colidx, values) or a
    torch sparse CSR tensor on the GPU; the latter is planned from device
    memory (sd_plan_device), its int64 indices narrowed to int32."""

    def __init__(self, A, widths, **plan_opts):
        self.plans = {}
        if isinstance(A, torch.Tensor):
            if A.layout != torch.sparse_csr or not A.is_cuda or A.dtype != torch.float32:
                raise ValueError("adjacency tensor must be a float32 sparse CSR tensor on the GPU")
            m, k = A.shape
            rowptr = A.crow_indices().to(torch.int32).contiguous()
            colidx = A.col_indices().to(torch.int32).contiguous()
            values = A.values().contiguous()
            stream = torch.cuda.current_stream(A.device)
            nnz = int(values.numel())

            def plan(n, **kw):
                return sd_plan_device(rowptr, colidx, values, m, k, nnz, n, stream=stream, **plan_opts, **kw)
        else:
            def plan(n, **kw):
                return sd_plan_ex(A, n, **plan_opts, **kw)
        for n in widths:
            self.plans[n] = (plan(n), plan(n, transpose=True))

    def __call__(self, B: torch.Tensor) -> torch.Tensor:
        fwd, bwd = self.plans[B.shape[1]]
        return spmm(B, fwd, bwd)

    def destroy(self):
        for fwd, bwd in self.plans.values():
            fwd.destroy()
            bwd.destroy()
        self.plans = {}


class GCN2(torch.nn.Module):
    """H1 = relu(Â X W1), logits = Â H1 W2 (transform, then aggregate)."""

    def __init__(self, A, in_feats: int, hidden: int, classes: int, device, seed: int = 0, **plan_opts):
        super().__init__()
        g = torch.Generator(device="cpu").manual_seed(seed)

        def glorot(fan_in, fan_out):
            bound = (6.0 / (fan_in + fan_out)) ** 0.5
            return (torch.rand((fan_in, fan_out), generator=g, dtype=torch.float32) * 2 - 1) * bound

        self.W1 = torch.nn.Parameter(glorot(in_feats, hidden).to(device))
        self.W2 = torch.nn.Parameter(glorot(hidden, classes).to(device))
        self.agg = AggregationPlans(A, sorted({hidden, classes}), **plan_opts)

    def forward(self, X: torch.Tensor) -> torch.Tensor:
        H1 = torch.relu(self.agg(transform(X, self.W1)))
        return self.agg(transform(H1, self.W2))


def train_epoch(model: GCN2, X, labels, opt) -> torch.Tensor:
    """One full-batch epoch: forward, cross-entropy, backward, optimiser step."""
    opt.zero_grad(set_to_none=True)
    loss = torch.nn.functional.cross_entropy(model(X), labels)
    loss.backward()
    opt.step()
    return loss.detach()
