"""Subdomain hops in launches past the sizes up to which other kernels take
them: every instance of the wavefront kernel, on 256 subdomains of 2 x 6 x 10 x
2 whose three regions end in the middle of a block of 16 sites (120, 424 and 984 sites), through one operator application
and, with the fused dot, through the inner CG.

A few subdomains stand for all (they do not touch each other), the first and
the last among them.  Bounds: FP32 1e-6, the bound of an FP32 operator
application; FP16 and INT8 2.5 times the error the format itself causes on this
input (the oracle's model of the stored fields) plus 1e-3 for the
epilogue's FP16 operands, each within 2^-12 of its site column's largest
value, per operator application.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

DIMS, SUB = (16, 12, 20, 16), (2, 6, 10, 2)


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def setup(Ls, prec, dims=DIMS, sub=SUB):
    from paper_2104_05615_amd import MSPCG
    U = W.gauge_field(dims, 0.5, 61)
    op = oracle.MobiusDWF(U, Ls, 1.5, 0.5, 1.8, 0.1)
    held = oracle.MobiusDWF(oracle.stored_links(U, prec), Ls, 1.5, 0.5, 1.8, 0.1)
    til = oracle.Tiling(dims, sub)
    g = np.random.default_rng(62).standard_normal((Ls, op.vh, 4, 3, 2))
    s = MSPCG(dims)
    s.load_gauge(U)
    s.set_mobius(Ls, 1.5, 0.5, 1.8, 0.1)
    s.set_subdomains(sub)
    return s, op, held, til, g[..., 0] + 1j * g[..., 1], [0, til.nsub // 3, til.nsub - 1]


PAST = [(p, Ls, DIMS, SUB) for p in ("fp32", "fp16", "int8") for Ls in (4, 8, 12, 16)]
# INT8 with Ls 12 below and at its two limits: 384 blocks in h1 and h3; 768 in them; 1024 in h4
EDGE = [("int8", 12, dims, (4, 4, 4, 4)) for dims in ((8, 8, 8, 8), (8, 8, 8, 16), (16, 16, 16, 8))]


@pytest.mark.parametrize("prec,Ls,dims,sub", PAST + EDGE)
def test_local_operator_past_the_launch_limit(prec, Ls, dims, sub):
    s, op, held, til, r, few = setup(Ls, prec, dims, sub)
    vs = np.stack([r[:, til.index[d]] for d in few])
    exact = oracle.local_operator(op, til, vs, subset=few, padded=True)
    tol = 1e-6
    if prec != "fp32":
        tol = 2.5 * rel(oracle.local_operator_stored(held, til, vs, prec, subset=few), exact) + 1e-3
    out = s.apply("A_sub", prec, r)
    got = np.stack([out[:, til.index[d]] for d in few])
    worst = max(rel(got[j], exact[j]) for j in range(len(few)))
    print(f"[gpu] A_sub {prec} Ls={Ls} dims={dims}: {worst:.2e}, bound {tol:.2e}", flush=True)
    assert worst < tol
    # no site of any subdomain is left out
    assert np.all(np.abs(out).max(axis=(0, 2, 3)) > 0)


@pytest.mark.parametrize("Ls", [8, 12, 16])
def test_preconditioner_past_the_launch_limit(Ls):
    k, prec = 2, "int8"
    s, op, held, til, r, few = setup(Ls, prec)
    s.set_solver(inner_iters=k)
    exact = oracle.inner_cg(op, til, r, k, subset=few, padded=True)
    tol = 2.5 * rel(oracle.inner_cg_stored(held, til, r, k, prec, subset=few), exact) + 1e-3 * k
    out = s.apply("precond", prec, r)
    got = np.stack([out[:, til.index[d]] for d in few])
    worst = max(rel(got[j], exact[j]) for j in range(len(few)))
    print(f"[gpu] precond {prec} Ls={Ls} k={k}: {worst:.2e}, bound {tol:.2e}", flush=True)
    assert worst < tol
