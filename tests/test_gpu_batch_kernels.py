"""A batched launch has the blocks of all its right-hand sides, so its subdomain
hops can run on another kernel than those of a single solve (the one with a
lane per 5D site and the general one for small launches, the one with a
wavefront per 16 sites past them).  All of them return the same bits, and with
them a batched solve those of its single solves.  At 8^4 with 4^4 subdomains
some of the four hops of 13 sources (h1 in every case) run on another kernel
than those of one.  A few iterations, each with two inner steps, on both sides.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DIMS, SUB, NRHS = (8, 8, 8, 8), (4, 4, 4, 4), 13


@pytest.mark.parametrize("inner,Ls", [("fp16", 4), ("fp16", 8), ("fp16", 16), ("int8", 8), ("int8", 12),
                                      ("int8", 16), ("fp32", 8)])
def test_batch_equals_single_solves_across_kernels(inner, Ls):
    import torch
    from paper_2104_05615_amd import MSPCG
    s = MSPCG(DIMS)
    s.load_gauge(W.gauge_field(DIMS, 0.5, 71))
    s.set_mobius(Ls, 1.5, 0.5, 1.8, 0.05)
    s.set_subdomains(SUB)
    s.set_solver(tol=1e-10, maxiter=3, inner_iters=2, inner_prec=inner, outer_prec="fp32")
    vh = int(np.prod(DIMS)) // 2
    b = torch.from_numpy(np.random.default_rng(72).standard_normal((NRHS, Ls, vh, 4, 3, 2))).cuda()
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    print(f"[gpu] {NRHS} RHS inner={inner} Ls={Ls}", flush=True)
    s.solve_batch_device(NRHS, b.data_ptr(), x.data_ptr())
    torch.cuda.synchronize()
    assert bool((x.abs().amax(dim=(1, 2, 3, 4, 5)) > 0).all())
    for i in (0, 6, NRHS - 1):
        x1 = torch.zeros_like(b[i])
        torch.cuda.synchronize()
        s.solve_device(b[i].data_ptr(), x1.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(x[i], x1)
