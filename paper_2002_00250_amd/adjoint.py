"""GMM adjoint over a window of frames, as a torch.autograd.Function.

``GmmWindowFunction.apply(theta, rgb, depth, window)`` returns the pre-update scores
Z [T, H, W] (float32) and the term flags [T, H, W] (uint8) of a fresh RGB-D GMM run over
the window; its backward returns dL/dtheta for theta = (alpha, lambda, w_depth), with the
forward's discrete choices held fixed.  Both directions run in libfgs kernels
(fgs_gmm_window_forward / _backward); this module only orders them on torch streams.
"""
from __future__ import annotations

import numpy as np
import torch
from torch.overrides import _get_current_function_mode_stack
from torch.utils._device import DeviceContext

from . import fgs


class GmmWindow:
    """Device buffers (records, checkpoints, scratch) for T frames of H x W, bounded by
    ``checkpoint_every`` (fgs_gmm_window_create).  The records and checkpoints belong to the most
    recent forward; ``forwards`` counts them."""

    def __init__(self, T: int, H: int, W: int, params=None, checkpoint_every: int = 16, device=None):
        self.T, self.H, self.W = T, H, W
        self.forwards = 0
        self.device = torch.device(device or "cuda")
        self.stream = torch.cuda.Stream(self.device)
        self.handle = fgs.fgs_gmm_window_create(T, H, W, params, checkpoint_every, self.stream.cuda_stream)
        with torch.cuda.device(self.device):
            self._order = fgs.StreamOrder(self.stream.cuda_stream)

    def close(self):
        if getattr(self, "handle", None):
            self._order.close()
            fgs.fgs_gmm_window_destroy(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, rgb, depth):
        T, H, W = self.T, self.H, self.W
        if tuple(rgb.shape) != (T, H, W, 3) or rgb.dtype != torch.uint8 or not rgb.is_contiguous():
            raise ValueError("rgb must be a contiguous uint8 tensor [T, H, W, 3]")
        if tuple(depth.shape) != (T, H, W) or depth.dtype not in (torch.int16, torch.uint16) \
                or not depth.is_contiguous():
            raise ValueError("depth must be a contiguous 16-bit tensor [T, H, W]")

    @staticmethod
    def _used_on(cur, *tensors):
        """`cur`, the current stream, waits for the window's from here on, so that memory taken from it
        is reused only behind the kernel.  A tensor made on another stream is marked as used on `cur`:
        its own stream does not wait for the kernel."""
        for x in tensors:
            x.record_stream(cur)              # (nothing to do for a tensor of `cur` itself)

    def forward(self, theta: torch.Tensor, rgb: torch.Tensor, depth: torch.Tensor):
        self._check(rgb, depth)
        theta = theta.detach().to(torch.float32).contiguous()
        cur = torch.cuda.current_stream(self.device)
        Z = torch.empty((self.T, self.H, self.W), dtype=torch.float32, device=self.device)
        has = torch.empty((self.T, self.H, self.W), dtype=torch.uint8, device=self.device)
        self._order.enter(cur)
        fgs.fgs_gmm_window_forward(self.handle, theta.data_ptr(), rgb.data_ptr(), depth.data_ptr(),
                                   Z.data_ptr(), has.data_ptr())
        self._order.leave(cur)
        self._used_on(cur, theta, rgb, depth)
        self.forwards += 1
        return Z, has

    def backward(self, theta: torch.Tensor, rgb: torch.Tensor, depth: torch.Tensor, dZ: torch.Tensor):
        self._check(rgb, depth)
        theta = theta.detach().to(torch.float32).contiguous()
        dZ = dZ.detach().to(torch.float32).contiguous()
        cur = torch.cuda.current_stream(self.device)
        out = torch.empty(3, dtype=torch.float64, device=self.device)
        self._order.enter(cur)
        fgs.fgs_gmm_window_backward(self.handle, theta.data_ptr(), rgb.data_ptr(), depth.data_ptr(),
                                    dZ.data_ptr(), out.data_ptr())
        self._order.leave(cur)
        self._used_on(cur, theta, rgb, depth, dZ)
        return out

    def records(self) -> np.ndarray:
        out = np.empty((self.T, self.H, self.W), np.uint64)
        torch.cuda.current_stream(self.device).synchronize()
        fgs.fgs_gmm_window_records(self.handle, out.ctypes.data, fgs.FGS_MEM_HOST)
        return out


class GmmWindowFunction(torch.autograd.Function):
    """Z, has = apply(theta, rgb, depth, window).  Several applications may share a window
    (two windows of a sequence in one loss, a probe at another theta): the backward of an
    application whose records a later forward has overwritten first runs its own forward
    again on the saved inputs (the same kernels, so the same records), then the adjoint."""

    @staticmethod
    def forward(ctx, theta, rgb, depth, window: GmmWindow):
        Z, has = window.forward(theta, rgb, depth)
        ctx.save_for_backward(theta, rgb, depth)
        ctx.window = window
        ctx.forward_id = window.forwards
        ctx.mark_non_differentiable(has)
        return Z, has

    @staticmethod
    def backward(ctx, gZ, ghas):
        theta, rgb, depth = ctx.saved_tensors
        if ctx.window.forwards != ctx.forward_id:
            ctx.window.forward(theta, rgb, depth)
            ctx.forward_id = ctx.window.forwards
        d = ctx.window.backward(theta, rgb, depth, gZ)
        return d.to(theta.dtype), None, None, None


def _bce_torch(Z, has, gt, t0, tau):
    w = has[t0:].to(Z.dtype)
    y = (gt[t0:] != 0).to(Z.dtype)
    l = torch.nn.functional.binary_cross_entropy_with_logits(Z[t0:] / tau, y, weight=w, reduction="sum")
    return l / w.sum().clamp_min(1.0)


def _watched() -> bool:
    """Whether something follows the operations themselves, which a kernel launched on raw pointers
    does not show: the function transforms, forward-mode differentiation, tracing, compiling, and
    Python dispatch and function modes (make_fx traces real tensors through them; a default device,
    which is such a mode too, only places new tensors)."""
    return (torch._C._are_functorch_transforms_active() or torch.autograd.forward_ad._current_level >= 0 or
            torch.jit.is_tracing() or torch.compiler.is_compiling() or torch._C._len_torch_dispatch_stack() > 0 or
            torch._C._len_torch_function_stack() > 0 and
            any(type(m) is not DeviceContext for m in _get_current_function_mode_stack()))


def _bce_kernel_takes(Z, has, gt, t0, tau) -> bool:
    """Whether the library's loss kernels compute this call: dense tensors of one shape on the
    current GPU (float32 scores, uint8 flags, uint8 or bool truth), plain numbers t0 and tau, and
    nothing watching the operations, which only the composed form answers."""
    if not (type(Z) in (torch.Tensor, torch.nn.Parameter) and type(has) is torch.Tensor and type(gt) is torch.Tensor):
        return False
    if not (Z.is_cuda and Z.dtype == torch.float32 and has.dtype == torch.uint8 and
            gt.dtype in (torch.uint8, torch.bool) and Z.device == has.device == gt.device and
            Z.device.index == torch.cuda.current_device()):
        return False
    if type(t0) is not int or type(tau) not in (int, float) or Z.dim() < 1 or not 0 <= t0 < Z.shape[0]:
        return False
    if Z.numel() == 0 or Z.shape != has.shape or Z.shape != gt.shape or Z.layout != torch.strided or \
            not (Z.is_contiguous() and has.is_contiguous() and gt.is_contiguous()):
        return False
    return not _watched()


def _bce_forward(Z, has, gt, t0, tau, keep):
    """The loss and, to keep, the slopes, the weights and the sums."""
    loss = torch.empty((), dtype=torch.float32, device=Z.device)
    work = torch.empty(fgs.FGS_WINDOW_BCE_WORK, dtype=torch.float64, device=Z.device)
    i0 = t0 * (Z.numel() // Z.shape[0])
    args = Z.data_ptr(), has.data_ptr(), gt.data_ptr(), i0, Z.numel(), tau, work.data_ptr(), loss.data_ptr()
    stream = torch.cuda.current_stream(Z.device).cuda_stream
    if not keep:
        fgs.fgs_window_bce(*args, stream)
        return loss
    slope, weight = torch.empty_like(Z), torch.empty_like(has)
    fgs.fgs_window_bce_keep(*args, slope.data_ptr(), weight.data_ptr(), stream)
    return loss, slope, weight, work, i0


class _WindowBce(torch.autograd.Function):
    """loss, slope = apply(Z, has, gt, t0, tau): the loss in one pass over the scores, which keeps its
    slope (sigmoid(Z / tau) - y) w for the gradient's pass.  Nothing of Z, has and gt is kept: the
    caller may refill them before the backward.  The slope is an output so that a gradient can be
    differentiated again (its own slope is p (1 - p) w / tau, p = |slope| / w)."""

    @staticmethod
    def forward(ctx, Z, has, gt, t0, tau):
        loss, slope, weight, work, i0 = _bce_forward(Z, has, gt, t0, tau, True)
        ctx.save_for_backward(slope, weight, work)
        ctx.i0, ctx.tau, ctx.device = i0, tau, Z.device
        ctx.set_materialize_grads(False)
        return loss, slope

    @staticmethod
    def backward(ctx, g, g_slope):
        slope, weight, work = ctx.saved_tensors
        if g is not None and g_slope is None and _kept_kernel_takes(ctx, g, slope, work):
            dZ = torch.empty_like(slope)
            fgs.fgs_window_bce_kept_grad(slope.data_ptr(), ctx.i0, slope.numel(), ctx.tau, work.data_ptr(),
                                         g.data_ptr(), dZ.data_ptr(),
                                         torch.cuda.current_stream(dZ.device).cuda_stream)
            return dZ, None, None, None, None
        # a gradient that is itself differentiated, or batched, or watched
        dZ = None
        if g is not None:
            dZ = slope * (g / work[1].to(g.dtype)) / ctx.tau
        if g_slope is not None:
            d = g_slope * (slope.abs() - slope * slope / weight.clamp(min=1)) / ctx.tau
            dZ = d if dZ is None else dZ + d
        return dZ, None, None, None, None


def _kept_kernel_takes(ctx, g, slope, work) -> bool:
    """Whether the library's gradient kernel computes this backward: a plain gradient (a batch of
    gradients has no storage of its own) and what the forward kept, as it was (a saved-tensor hook
    may give back something else), on the current GPU."""
    def same(x, dtype):
        return type(x) is torch.Tensor and x.device == ctx.device and x.dtype == dtype and x.is_contiguous() and \
            torch._C._has_storage(x)
    return ctx.device.index == torch.cuda.current_device() and not torch.is_grad_enabled() and not _watched() and \
        same(g, torch.float32) and g.numel() == 1 and same(slope, torch.float32) and \
        same(work, torch.float64) and work.numel() == fgs.FGS_WINDOW_BCE_WORK


def window_bce_loss(Z: torch.Tensor, has: torch.Tensor, gt: torch.Tensor, t0: int = 1, tau: float = 1.0):
    """Mean BCE of sigmoid(Z/tau) against 0/255 ground truth over frames t >= t0 where Z has a term."""
    if not _bce_kernel_takes(Z, has, gt, t0, tau):
        return _bce_torch(Z, has, gt, t0, tau)
    if torch.is_grad_enabled() and Z.requires_grad:
        return _WindowBce.apply(Z, has, gt, t0, tau)[0]
    return _bce_forward(Z, has, gt, t0, tau, False)
