"""Subdomain hops of the 16- and 8-bit formats on both sides of the launch size
from which other kernels than the one with a lane per 5D site take them (the
lattices put a hop at that size exactly and others past it; ragged tilings of
small lattices are in test_gpu_wave_hops), and NaN in its packed epilogue.

Bounds: 2.5 times the error the format itself causes on this input (the
oracle's model of the stored fields) plus 1e-3 for the epilogue's FP16
operands, each within 2^-12 of its site column's largest value.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def setup(dims, Ls, sub, seed):
    from paper_2104_05615_amd import MSPCG
    U = W.gauge_field(dims, 0.5, seed)
    s = MSPCG(dims)
    s.load_gauge(U)
    s.set_mobius(Ls, 1.5, 0.5, 1.8, 0.1)
    s.set_subdomains(sub)
    vh = int(np.prod(dims)) // 2
    g = np.random.default_rng(seed + 1).standard_normal((Ls, vh, 4, 3, 2))
    return s, U, g[..., 0] + 1j * g[..., 1]


@pytest.mark.parametrize("dims,Ls", [((16, 16, 16, 8), 4), ((8, 8, 16, 16), 8), ((8, 8, 8, 16), 16),
                                     ((8, 8, 16, 16), 16)])
def test_local_operator_across_launch_sizes(dims, Ls):
    sub = (4, 4, 4, 4)
    s, U, r = setup(dims, Ls, sub, 51)
    op = oracle.MobiusDWF(U, Ls, 1.5, 0.5, 1.8, 0.1)
    til = oracle.Tiling(dims, sub)
    few = [0, 7, til.nsub - 1]   # subdomains do not touch each other: these stand for all
    vs = np.stack([r[:, til.index[d]] for d in few])
    exact = oracle.local_operator(op, til, vs, subset=few)
    for prec in ("fp16", "int8"):
        held = oracle.MobiusDWF(oracle.stored_links(U, prec), Ls, 1.5, 0.5, 1.8, 0.1)
        tol = 2.5 * rel(oracle.local_operator_stored(held, til, vs, prec, subset=few), exact) + 1e-3
        out = s.apply("A_sub", prec, r)
        e = rel(np.stack([out[:, til.index[d]] for d in few]), exact)
        print(f"[gpu] A_sub {prec} dims={dims} Ls={Ls}: {e:.2e}, bound {tol:.2e}", flush=True)
        assert e < tol


@pytest.mark.parametrize("Ls", [4, 8, 16])
def test_nan_stays_at_the_sites_that_read_it(Ls):
    dims, sub = (2, 6, 24, 2), (2, 2, 12, 2)
    s, _, r = setup(dims, Ls, sub, 53)
    r[:, oracle.Tiling(dims, sub).index[1][0]] = np.nan
    want = np.isnan(s.apply("A_sub", "fp32", r))
    got = np.isnan(s.apply("A_sub", "fp16", r))
    assert want.any() and not want.all()
    assert np.array_equal(got, want)
