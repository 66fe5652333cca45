"""Training a dual-domain two-mask receiver through turbulence (Sec. 2.5, Sec. 4).

Each epoch propagates a batch through fresh screens (time index = epoch) with
the fused GPU path, applies the receiver with the two learnable masks, and
minimises scintillation inside the aperture plus the L2 distance of the mean
intensity to the vacuum beam through the same receiver:

    L = sum_A Var_b(I) / sum_A (E_b I)^2 + sum (E_b I - I_vac)^2 / sum I_vac^2

with Adam and a one-cycle learning-rate schedule from a constant (zero) phase
initialisation (Sec. 2.5).  Propagation, receiver and loss (forward and adjoint) run in
libturpy.
"""

import numpy as np
import torch

from . import api
from . import binding as B


class _Loss(torch.autograd.Function):
    """The loss and its gradient in two passes over the fields
    (turpy_receiver_loss).  The forward pass leaves its sums and, behind them,
    the mean intensities in one buffer."""

    SUMS = 4 + 4 * 1024

    @staticmethod
    def forward(ctx, u_out, i_vac, aperture):
        pixels, batch = i_vac.numel(), u_out.shape[0]
        work = torch.empty(_Loss.SUMS + (pixels + 1) // 2, dtype=torch.float64, device=u_out.device)
        loss = torch.empty((), dtype=torch.float32, device=u_out.device)
        sums = work.data_ptr()
        B.receiver_loss(pixels, batch, u_out.data_ptr(), i_vac.data_ptr(), aperture.data_ptr(), sums + 8 * _Loss.SUMS,
                        sums, loss.data_ptr(), _stream(u_out))
        ctx.save_for_backward(u_out, i_vac, aperture, work)
        return loss

    @staticmethod
    def backward(ctx, grad_loss):
        u_out, i_vac, aperture, work = ctx.saved_tensors
        if torch.is_grad_enabled():  # create_graph: a gradient that can be differentiated again
            return torch.autograd.grad(_loss_ops(u_out, i_vac, aperture), u_out, grad_loss, create_graph=True) + \
                (None, None)
        # batched cotangents (vmap over the backward pass) have no memory of their own, and a
        # dual one has a tangent to carry: the kernel then takes 1, and tensor operations the rest
        direct = torch._C._has_storage(grad_loss) and not _dual(grad_loss)
        # saved-tensor hooks may hand back other types and layouts than were saved
        if _readable(u_out, i_vac, aperture) and _plain(work) and work.dtype is torch.float64 and \
                work.device == u_out.device and work.numel() == _Loss.SUMS + (i_vac.numel() + 1) // 2 and \
                work.is_contiguous():
            unit = grad_loss.resolve_neg() if direct else torch.ones((), dtype=torch.float32, device=u_out.device)
            grad_u = torch.empty_like(u_out)
            sums = work.data_ptr()
            B.receiver_loss_backward(i_vac.numel(), u_out.shape[0], u_out.data_ptr(), i_vac.data_ptr(),
                                     aperture.data_ptr(), sums + 8 * _Loss.SUMS, sums, unit.data_ptr(),
                                     grad_u.data_ptr(), _stream(u_out))
            if direct:
                return grad_u, None, None
        else:
            with torch.enable_grad():
                u_again = u_out.detach().requires_grad_()
                (grad_u,) = torch.autograd.grad(_loss_ops(u_again, i_vac, aperture), u_again)
        return grad_u * grad_loss, None, None


def _stream(t):
    return torch._C._cuda_getCurrentRawStream(t.device.index)


_PLAIN = (torch.Tensor, torch.nn.Parameter)


def _plain(t):
    return type(t) in _PLAIN and not t.is_neg() and not _dual(t)


def _dual(t):
    """Whether t carries a forward-mode tangent."""
    ad = torch.autograd.forward_ad
    return ad._current_level >= 0 and ad.unpack_dual(t).tangent is not None


def _readable(u_out, i_vac, aperture):
    """Whether the library's kernels can read these: contiguous complex64 fields
    and float32 planes on the current GPU, within the sizes they take."""
    if not (_plain(u_out) and _plain(i_vac) and _plain(aperture) and u_out.is_cuda):
        return False
    shape, device, f32 = u_out.shape, u_out.device, torch.float32
    return (len(shape) == 3 and i_vac.shape == shape[1:] and aperture.shape == i_vac.shape
            and 0 < shape[0] <= 1 << 19 and 0 < i_vac.numel() <= 1 << 32
            and u_out.dtype is torch.complex64 and i_vac.dtype is f32 and aperture.dtype is f32
            and i_vac.device == device and aperture.device == device and device.index == torch.cuda.current_device()
            and u_out.is_contiguous() and i_vac.is_contiguous() and aperture.is_contiguous() and not u_out.is_conj())


def _fused(u_out, i_vac, aperture):
    """Whether the library's kernels can stand in for the tensor operations:
    inputs they can read, no gradient asked for the planes, and nobody watching
    the operations (function transforms, forward-mode derivatives, tracing,
    compilation, tensor subclasses)."""
    if torch._C._are_functorch_transforms_active() or torch.jit.is_tracing() or torch.compiler.is_compiling():
        return False
    if torch.overrides._get_current_function_mode_stack() or torch.utils._python_dispatch._get_current_dispatch_mode():
        return False
    return not (i_vac.requires_grad or aperture.requires_grad) and _readable(u_out, i_vac, aperture)


def loss_fn(u_out, i_vac, aperture):
    return (_Loss.apply if _fused(u_out, i_vac, aperture) else _loss_ops)(u_out, i_vac, aperture)


def _loss_ops(u_out, i_vac, aperture):
    inten = u_out.real ** 2 + u_out.imag ** 2
    m1 = inten.mean(0)
    var = ((inten - m1) ** 2).mean(0)
    l_si = (var * aperture).sum() / ((m1 * m1) * aperture).sum()
    l_l2 = ((m1 - i_vac) ** 2).sum() / (i_vac * i_vac).sum()
    return l_si + l_l2


def aperture_mask(n, dx, diameter, device):
    x = (torch.arange(n, dtype=torch.float64, device=device) - n // 2) * dx
    return ((x[None, :] ** 2 + x[:, None] ** 2) <= (0.5 * diameter) ** 2).to(torch.float32)


class D2NNTrainer:
    def __init__(self, workload, diameter=0.3048, lr=0.01, epochs=100, device="cuda"):
        p = workload.path
        self.w, self.path = workload, p
        self.plan = api.Plan(p)
        self.rx = api.Receiver(p.n, p.dx, diameter)
        self.u0 = torch.from_numpy(workload.source_field().astype(np.complex64)).to(device)
        vac = api.Plan(p.with_(cn2dz=tuple(0.0 for _ in p.cn2dz), realizations=1))
        zero = torch.zeros((p.n, p.n), dtype=torch.float32, device=device)
        u_vac = self.rx.forward(vac.propagate(self.u0), zero, zero)
        self.i_vac = (u_vac.real ** 2 + u_vac.imag ** 2)[0]
        vac.close()
        self.aperture = aperture_mask(p.n, p.dx, diameter, device)
        self.theta1 = torch.zeros((p.n, p.n), dtype=torch.float32, device=device, requires_grad=True)
        self.theta2 = torch.zeros((p.n, p.n), dtype=torch.float32, device=device, requires_grad=True)
        self.opt = torch.optim.Adam([self.theta1, self.theta2], lr=lr)
        self.sched = torch.optim.lr_scheduler.OneCycleLR(self.opt, max_lr=lr, total_steps=epochs)

    def forward(self, epoch):
        u_rx = api.Propagate.apply(self.u0, None, self.plan, self.w.seed, epoch)
        return api.ReceiverFn.apply(u_rx, self.theta1, self.theta2, self.rx)

    def step(self, epoch):
        self.opt.zero_grad(set_to_none=True)
        loss = loss_fn(self.forward(epoch), self.i_vac, self.aperture)
        loss.backward()
        self.opt.step()
        self.sched.step()
        return loss.detach()
