"""More calls for the LDS-poison check, at the sizes that lds_poison_cases.py
leaves to the one-wave-per-transform row schedule: the relay and pair schedules
at every grid size they are built for, single realizations, groups past the
one-wave line, screens given by the caller, the other radix plan, lean column
strips, and the training loss.  Outputs are kept as SHA-256 digests.  Run as a
script: python lds_poison_schedules.py OUT.npz."""
import hashlib
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
for _d in (ROOT, HERE):
    if _d not in sys.path:
        sys.path.insert(0, _d)

from lds_poison_cases import _path  # noqa: E402


def run_cases():
    """{name: uint8 digest, or zeros where an output is not finite}."""
    import torch

    from paper_2604_07248_amd import api, binding, d2nn, workloads
    binding.lib()
    out = {}

    def keep(name, t):
        torch.cuda.synchronize()
        a = t.detach().cpu().numpy()
        d = hashlib.sha256(np.ascontiguousarray(a).tobytes()).digest() if np.isfinite(a).all() else bytes(32)
        out[name] = np.frombuffer(d, dtype=np.uint8)
        print(f"[poison] {name}", file=sys.stderr, flush=True)

    def c64(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.complex64)).cuda()

    def every_call(name, plan, n, r, dx):
        u0 = c64(workloads.gaussian_source(n, dx, 0.1 * n * dx))
        keep(f"{name}_fwd", plan.propagate(u0, seed=5))
        o, ck = plan.propagate(u0, seed=5, checkpoints=True)
        keep(f"{name}_ck", ck)
        for kind, args, kw in (("bwd", (o, ck), {}), ("rev", (o, None), {"u_out": o})):
            g_in, g_phi = plan.propagate_backward(*args, seed=5, **kw)
            keep(f"{name}_{kind}_in", g_in)
            keep(f"{name}_{kind}_phi", g_phi)

    # above the one-wave line, an odd count among them; 2048 with lean strips
    for n, r, sh, tf in ((64, 515, 3, 0), (128, 130, 0, 1), (256, 34, 3, 0), (512, 11, 2, 0), (1024, 4, 0, 1),
                         (2048, 3, 3, 0)):
        p = _path(workloads, n, 2, r, sh, tf)
        plan = api.Plan(p)
        every_call(f"n{n}", plan, n, r, p.dx)
        if n in (512, 1024):
            plan.set_config(col_radix=4, synth_radix=4, ar_radix=4)
            every_call(f"n{n}_radix4", plan, n, r, p.dx)
        plan.close()
    # a single realization: real screens, and full planes kept with the checkpoints
    for n in (32, 64, 256, 1024, 2048):
        p = _path(workloads, n, 3, 1, 3)
        for flags in (0, binding.SCREEN_CHECKPOINTS):
            plan = api.Plan(p, flags=flags)
            every_call(f"one{n}_{flags}", plan, n, 1, p.dx)
            state = plan.init_spectra(7)
            u0 = c64(workloads.gaussian_source(n, p.dx, 0.1 * n * p.dx))
            keep(f"one{n}_{flags}_ar", plan.evolve_propagate(state, 7, 1, 0.95, 0.3, -0.2, u_in=u0))
            keep(f"one{n}_{flags}_state", state)
            plan.close()
    # screens given by the caller
    for n, r in ((32, 3), (256, 5)):
        p = _path(workloads, n, 2, r)
        plan = api.Plan(p)
        phi = plan.screens(seed=3)
        u0 = c64(workloads.gaussian_source(n, p.dx, 0.1 * n * p.dx))
        o, ck = plan.propagate(u0, seed=3, screens=phi, checkpoints=True)
        keep(f"given{n}", o)
        g_in, g_phi = plan.propagate_backward(o, ck, seed=3, screens=phi)
        keep(f"given{n}_in", g_in)
        keep(f"given{n}_phi", g_phi)
        plan.close()
    # groups past the line: 40 single realizations, 9 triples
    for name, paths in (("solo", [_path(workloads, 256, 1 + i % 3, 1, 3) for i in range(40)]),
                        ("pairs", [_path(workloads, 512, 1 + i % 2, 3) for i in range(9)])):
        batch = api.Batch(paths)
        src = batch.pack([c64(workloads.gaussian_source(q.n, q.dx, 0.1 * q.n * q.dx))
                          .expand(q.realizations, q.n, q.n) for q in paths])
        keep(f"group_{name}", batch.propagate(src, seed=3))
        bo, bck = batch.propagate(src, seed=3, checkpoints=True)
        keep(f"group_{name}_ck", bck)
        bg, bphi = batch.propagate_backward(bo, bck, seed=3)
        keep(f"group_{name}_in", bg)
        keep(f"group_{name}_phi", bphi)
        batch.close()
    # the training loss, with blocks of part and of several sweeps of pixels
    for b, n in ((3, 17), (17, 600)):
        g = torch.Generator(device="cuda").manual_seed(b)
        u = torch.randn((b, n, n), generator=g, device="cuda", dtype=torch.complex64).requires_grad_()
        iv, ap = torch.rand((n, n), generator=g, device="cuda"), torch.ones((n, n), device="cuda")
        loss = d2nn.loss_fn(u, iv, ap)
        keep(f"loss{n}", loss)
        keep(f"loss{n}_grad", torch.autograd.grad(loss, u)[0])
    return out


if __name__ == "__main__":
    np.savez(sys.argv[1], **run_cases())
