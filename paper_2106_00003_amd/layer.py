"""PyTorch autograd front end of the library: U(theta) applied to a batch of column vectors as a
differentiable operation (the training use the paper targets: Section 1 and the problem statement of
Section 2 — "forward" builds or applies U, "backward" turns dL/dY into dL/dtheta).

Marshalling only.  forward() is one givens_forward / givens_build call; backward() is one
givens_backward call on the saved *output* (the reverse sweep undoes the rotations, so no
activations other than Y are kept).  For float32 the forward pass prepares the coefficient tables of both
sweep directions once (givens_prepare, where givens_prepare_pays) and the backward pass reuses them -- theta cannot
change in between; if another call on the stream has replaced the tables meanwhile, the backward pass falls back to
the plain call, which rebuilds them.  There is no CPU path: tensors must live on the GPU.
"""
from __future__ import annotations

import torch

from . import binding


def _plain(n: int, m) -> bool:
    """True when the unrestricted entry points cover the problem (even n, every pair free)."""
    return n % 2 == 0 and (m is None or m == n - 1)


def _prepare(th, n, m, want_backward: bool, B: int) -> int:
    """Token of the prepared tables of th (float32), or 0 when the prepared path does not apply."""
    if th.dtype != torch.float32 or B < 1 or not binding.givens_prepare_pays(n, m, B):
        return 0
    directions = binding.PREPARE_FORWARD
    if want_backward:
        # wide batches take the Gram form, which a token has to be prepared for
        directions |= binding.PREPARE_BACKWARD_WIDE if B >= 2 * (n + n % 2) else binding.PREPARE_BACKWARD
    return binding.givens_prepare(th, n, m, directions, batch=B)


def _backward(token, th, Y, g, m, need_dx):
    """dX, dtheta from the prepared tables when they are still there, else from the plain call."""
    if token:
        try:
            return binding.givens_backward_prepared(token, Y, g, th.numel(), want_dx=need_dx)
        except binding.GivensError as err:
            if err.code != binding.ERR_STALE:
                raise
    if m is None:
        return binding.givens_backward(th, Y, g, want_dx=need_dx)
    return binding.givens_backward_restricted(th, Y, g, m, want_dx=need_dx)


class _GivensApply(torch.autograd.Function):
    @staticmethod
    def forward(ctx, theta, X, m):
        th, x = theta.detach().contiguous(), X.detach().contiguous()
        n = x.shape[0]
        ctx.m = None if _plain(n, m) else (n - 1 if m is None else m)
        ctx.token = _prepare(th, n, ctx.m, any(ctx.needs_input_grad), x.shape[1])
        if ctx.token:
            Y = binding.givens_forward_prepared(ctx.token, x)
        else:
            Y = binding.givens_forward(th, x) if ctx.m is None else binding.givens_forward_restricted(th, x, ctx.m)
        ctx.save_for_backward(theta, Y)
        return Y

    @staticmethod
    @torch.autograd.function.once_differentiable
    def backward(ctx, G):
        theta, Y = ctx.saved_tensors
        need_dx = ctx.needs_input_grad[1]
        th, g = theta.detach().contiguous(), G.contiguous()
        dX, dtheta = _backward(ctx.token, th, Y, g, ctx.m, need_dx)
        return (dtheta if ctx.needs_input_grad[0] else None), (dX if need_dx else None), None


class _GivensMatrix(torch.autograd.Function):
    @staticmethod
    def forward(ctx, theta, n, m):
        th = theta.detach().contiguous()
        ctx.m = None if _plain(n, m) else (n - 1 if m is None else m)
        ctx.token = _prepare(th, n, ctx.m, ctx.needs_input_grad[0], n)
        if ctx.token:
            U = binding.givens_build_prepared(ctx.token, n, th.device)
        else:
            U = binding.givens_build(th, n) if ctx.m is None else binding.givens_build_restricted(th, n, ctx.m)
        ctx.save_for_backward(theta, U)
        return U

    @staticmethod
    @torch.autograd.function.once_differentiable
    def backward(ctx, G):
        theta, U = ctx.saved_tensors
        th, g = theta.detach().contiguous(), G.contiguous()
        _, dtheta = _backward(ctx.token, th, U, g, ctx.m, False)
        return dtheta, None, None


class _UnitaryApply(torch.autograd.Function):
    @staticmethod
    def forward(ctx, theta, phi, X):
        Y = binding.givens_unitary_forward(theta.detach().contiguous(), phi.detach().contiguous(),
                                           X.detach().contiguous())
        ctx.save_for_backward(theta, phi, Y)
        return Y

    @staticmethod
    @torch.autograd.function.once_differentiable
    def backward(ctx, G):
        # PyTorch hands a complex output's gradient over as dL/dRe + i dL/dIm for a real loss L, which is
        # the convention of givens_unitary_backward, and expects the same for the complex input X.
        theta, phi, Y = ctx.saved_tensors
        need_dx = ctx.needs_input_grad[2]
        dX, dtheta, dphi = binding.givens_unitary_backward(theta.detach().contiguous(), phi.detach().contiguous(),
                                                           Y, G.contiguous(), want_dx=need_dx)
        return dtheta, dphi, (dX if need_dx else None)


def givens_unitary_apply(theta: torch.Tensor, phi: torch.Tensor, X: torch.Tensor) -> torch.Tensor:
    """Y = U(theta, phi) X for complex X of shape (n, B) (the paper's appendix on U(n)); differentiable in
    theta, phi and X."""
    return _UnitaryApply.apply(theta, phi, X)


def givens_apply(theta: torch.Tensor, X: torch.Tensor, m: int | None = None) -> torch.Tensor:
    """Y = U(theta) X for X of shape (n, B) (columns are the batch); differentiable in theta and X.
    m restricts the parametrisation to the pairs (i, j) with i < m (Section 5); n may be odd."""
    return _GivensApply.apply(theta, X, m)


def givens_matrix(theta: torch.Tensor, n: int, m: int | None = None) -> torch.Tensor:
    """U(theta) itself, n x n; differentiable in theta."""
    return _GivensMatrix.apply(theta, n, m)


# Evaluation.  Building and laying out U costs as much as 1.5 plain calls with few columns up to n = 2048, two at 4096 and
# four at 8192 (B = 64: n = 1024 116 and 190 us, 2048 490 / 710, 4096 1190 / 2430, 8192 4.8 / 22 ms; below 512 host work
# decides, and a batch gains little by it).  So a layer whose last theta saw fewer batches than pay for a matrix (one batch
# per training step) evaluates the next one by plain calls.  The two differ in rounding, and batches of one theta should
# not differ with their number: a theta that is begun one way stays with it, up to a number of batches (times n / 2048)
# that only a layer in service again sees.  Up to n = 128 a plain call is as fast as a product with a kept matrix
# (n = 64, B = 64: 18 and 20 us).
_MATRIX_MIN_N = 129
_PLAIN_BATCHES = 32


def _worth_a_matrix(n: int) -> int:
    return 8 if n < 512 else max(2, n // 2048 + 1)


def _evaluate(th, x, m):
    """Y = U(th) x by a plain call."""
    n = x.shape[0]
    if _plain(n, m):
        return binding.givens_forward(th, x)
    return binding.givens_forward_restricted(th, x, n - 1 if m is None else m)


class _Run:
    """The batches evaluated with one theta (held, so that no other angles can come to lie at its address)."""

    def __init__(self, theta, plain):
        self.theta, self.version, self.plain, self.batches = theta, theta._version, plain, 0

    def of(self, theta) -> bool:
        return theta._version == self.version and theta.data_ptr() == self.theta.data_ptr()


class _KeptMatrix:
    """U of the present angles laid out for evaluation, for use on any stream: made on one, which others wait for."""

    def __init__(self, theta, th, n, m):
        self.theta, self.version, self.stream = theta, theta._version, binding.current_stream_key()
        U = binding.givens_build(th, n) if _plain(n, m) else binding.givens_build_restricted(th, n, n - 1 if m is None else m)
        self.matrix = binding.Kept(th, U, m)
        self.ready = torch.cuda.current_stream().record_event()

    def of(self, theta) -> bool:
        return theta._version == self.version and theta.data_ptr() == self.theta.data_ptr()

    def apply(self, th, x):
        if binding.current_stream_key() != self.stream:
            stream = torch.cuda.current_stream()
            stream.wait_event(self.ready)
            self.matrix.block.record_stream(stream)
        return binding.givens_apply_kept(self.matrix, th, x)


class OrthogonalLinear(torch.nn.Module):
    """Orthogonal layer y = U(theta) x on column batches (n, B), with the free angles as its parameters in
    the round-robin order E (Section 3): n(n-1)/2 of them, or m n - m(m+1)/2 with the parametrisation
    restricted to pairs (i, j), i < m (Section 5).  Angles start near zero (U near the identity)."""

    def __init__(self, n: int, m: int | None = None, init_std: float = 0.1, device="cuda", dtype=torch.float32):
        super().__init__()
        if n < 2:
            raise ValueError("n must be >= 2")
        self.n, self.m = n, m
        count = binding.num_angles(n, m)
        self.theta = torch.nn.Parameter(init_std * torch.randn(count, device=device, dtype=dtype))

        self._start_evaluation()

    def _start_evaluation(self) -> None:
        self._eval_matrix = None  # U laid out for evaluation, a _KeptMatrix
        self._eval_run = None     # the batches evaluated with the present theta, a _Run
        self._captured = []       # those that recorded graphs read

    def forward(self, X: torch.Tensor) -> torch.Tensor:
        theta = self.theta
        if torch.is_grad_enabled() or theta.dtype != torch.float32:
            return givens_apply(theta, X, self.m)
        x = X.contiguous()
        if x.dim() != 2 or x.shape[0] != self.n or x.shape[1] == 0 or x.dtype != torch.float32 or not x.is_cuda:
            return givens_apply(theta, X, self.m)   # refused there
        # evaluation: U of the current theta is built and laid out once, here and not in the workspace of the stream, which
        # all layers share, and multiplied with until theta changes.  The version counter tells most changes; writes that it
        # does not count (through .data, by a replayed graph) are seen on the device, which compares the angles.
        th = theta.contiguous()
        if self.n < _MATRIX_MIN_N:
            return _evaluate(th, x, self.m)
        kept = self._eval_matrix
        same = kept is not None and kept.of(theta)
        if torch.cuda.is_current_stream_capturing():
            if not same or kept.matrix.changed():
                return _evaluate(th, x, self.m)
            if not any(kept is k for k in self._captured):   # what a graph reads has to stay
                self._captured.append(kept)
            return binding.givens_apply_packed(kept.matrix.packed, x)
        run = self._eval_run
        if run is None or not run.of(theta) or (same and kept.matrix.changed()):
            # a new theta: by plain calls if the last one did not see enough batches to be worth a matrix
            run = self._eval_run = _Run(theta.detach(), run is not None and run.batches < _worth_a_matrix(self.n))
            same = False
        run.batches += 1
        if run.plain and run.batches <= _PLAIN_BATCHES * max(1, self.n // 2048):
            return _evaluate(th, x, self.m)
        if not same:
            self._eval_matrix = kept = _KeptMatrix(theta.detach(), th, self.n, self.m)
        try:
            return kept.apply(th, x)
        except binding.GivensError as err:
            if err.code != binding.ERR_STALE:      # (known to have changed by now: the next batch is a new theta's)
                raise
            return _evaluate(th, x, self.m)

    # what evaluation keeps stays with the object: a copy starts anew, from whichever version of this class it was pickled
    def __getstate__(self):
        return {k: v for k, v in self.__dict__.items() if k not in ("_eval_matrix", "_eval_run", "_captured")}

    def __setstate__(self, state):
        super().__setstate__({k: v for k, v in state.items() if k != "_eval_tables"})
        self._start_evaluation()

    def forget_recorded(self) -> None:
        """Gives up the matrices that graphs recorded in evaluation read (one for every theta that was recorded).  Only
        when none of these graphs is going to be replayed; without it they stay as long as the layer."""
        self._captured = []

    def matrix(self) -> torch.Tensor:
        return givens_matrix(self.theta, self.n, self.m)
