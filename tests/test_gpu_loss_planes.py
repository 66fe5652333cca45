"""The training loss on the largest plane it takes, 2^32 pixels: more than one
pixel for each thread a launch may have.  One field, zero but for a few pixels
on both sides of where a second sweep of the blocks begins, so that every sum
and gradient is known in closed form.  FP32 intensities carry 2^-23 relative:
1e-5."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_gradient_of_2_to_the_32_pixels(gpu_lib):
    from paper_2604_07248_amd import d2nn
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("needs 120 GB of free device memory")
    n = 1 << 16
    at = torch.tensor([0, 255, 256, 2 ** 31 + 5, 2 ** 32 - 513, 2 ** 32 - 257, 2 ** 32 - 256, 2 ** 32 - 1],
                      device="cuda")
    amp = torch.polar(torch.linspace(0.5, 2.0, len(at), device="cuda"), torch.linspace(-3, 3, len(at), device="cuda"))
    vac = torch.linspace(1.5, 0.2, len(at), device="cuda")
    u = torch.zeros((1, n, n), dtype=torch.complex64, device="cuda")
    iv, ap = torch.zeros((n, n), device="cuda"), torch.zeros((n, n), device="cuda")
    u.view(-1)[at], iv.view(-1)[at], ap.view(-1)[at] = amp, vac, torch.ones_like(vac)
    u.requires_grad_()
    assert d2nn._fused(u, iv, ap)
    loss = d2nn.loss_fn(u, iv, ap)
    (grad,) = torch.autograd.grad(loss, u)
    a, v = amp.to(torch.complex128).requires_grad_(), vac.double()
    ref = d2nn._loss_ops(a[None, None], v[None], torch.ones_like(v)[None])
    (want,) = torch.autograd.grad(ref, a)
    assert abs(float(loss) - float(ref)) <= 1e-5 * float(ref)
    got = grad.view(-1)[at].to(torch.complex128)
    assert torch.linalg.vector_norm(got - want) <= 1e-5 * torch.linalg.vector_norm(want)
    assert int(torch.count_nonzero(torch.view_as_real(grad))) == 2 * len(at)
    del u, iv, ap, grad
    torch.cuda.empty_cache()
