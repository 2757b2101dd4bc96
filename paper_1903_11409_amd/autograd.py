"""Autograd glue: the batched product as a differentiable PyTorch operation.

Argument marshalling only: the forward pass is one ``bspmm_run`` launch, the backward pass one
``bspmm_run_transposed`` launch on the same plan (the gradient with respect to the dense
operand, ``dB_i = A_i^T dY_i``; the adjacency values are constants of the layer, as in the
paper's graph-convolution layer, Sec. II-A / Sec. IV-D).
"""
import torch

from . import bspmm as K


def _output(plan, transposed, rows, device):
    """Room for a product.  The launch writes every row that belongs to an operation, so the rows
    are cleared first only when some belong to none (1024 graphs of 8 to 500 nodes at F = 256:
    clearing C and G took 16.8 us of a step's 71 us on the GPU)."""
    make = torch.empty if plan.covered_rows(transposed) >= rows else torch.zeros
    return make((rows, plan.F), dtype=torch.float32, device=device)


class BatchedSpMM(torch.autograd.Function):
    """``C = BatchedSpMM.apply(plan, B)`` with ``plan`` a :class:`bspmm.Plan`; ``B`` is the packed
    dense input (``n_b_rows x F`` fp32 on the plan's device), ``C`` the packed output."""

    @staticmethod
    def forward(ctx, plan, B, n_c_rows=None):
        if B.dtype != torch.float32 or not B.is_cuda:
            raise TypeError("BatchedSpMM needs an fp32 CUDA tensor")
        B = B.contiguous()
        rows = int(n_c_rows) if n_c_rows is not None else int(B.shape[0])
        C = _output(plan, False, rows, B.device)
        plan.run(B, C)
        ctx.plan = plan
        ctx.n_b_rows = int(B.shape[0])
        return C

    @staticmethod
    def backward(ctx, dY):
        dY = dY.contiguous()
        G = _output(ctx.plan, True, ctx.n_b_rows, dY.device)
        ctx.plan.run_transposed(dY, G)
        return None, G, None


class _Node(BatchedSpMM):
    """A node of the class without its product."""

    @staticmethod
    def forward(ctx, plan, B, n_c_rows):
        ctx.plan = plan
        ctx.n_b_rows = int(B.shape[0])
        return B.detach()[:1].expand(n_c_rows, plan.F)


def _node_of_class(plan, n_b_rows, n_c_rows):
    """A tensor whose node is the class's, for what traces the backward pass of a native one (compiled autograd)."""
    with torch.enable_grad():
        B = torch.empty((1, plan.F), dtype=torch.float32, device=plan.device).expand(n_b_rows, plan.F).requires_grad_()
        return _Node.apply(plan, B, n_c_rows)


def batched_spmm(plan: K.Plan, B, n_c_rows=None):
    """Functional form of :class:`BatchedSpMM`.  Rows of the output that belong to no operation
    are zero (``n_c_rows`` defaults to the number of rows of ``B``).

    Plain tensors take the same two steps in native code (csrc/binding.cpp): through the interpreter, which
    the engine's thread enters for the backward pass, a step of 47 graphs at F = 64 took the host 63 us, and takes
    23 to 43 now (1024 graphs of 8 to 500 nodes at F = 256: 63 -> 55, the time of the two launches).  What the native
    code leaves out - tensor subclasses, active modes, tracing, forward-mode gradients, function
    transforms - goes through the class, and compiled autograd finds the class's node in the native one."""
    if (type(plan) is K.Plan and not torch._C._are_functorch_transforms_active()
            and not torch.compiler.is_compiling()):
        C = K._native.batched_spmm(plan, plan.handle, plan.F, B, n_c_rows, _node_of_class)
        if C is not None:
            return C
    return BatchedSpMM.apply(plan, B, n_c_rows)
