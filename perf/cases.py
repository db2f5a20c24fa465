"""The work this library is given in practice, as cases that can be timed.

A program that uses the library holds a handle (gauge field, Moebius
parameters, subdomain tiling, solver parameters) and device buffers, and calls
three kinds of entry point on them: one operator or preconditioner application
(``apply_device``; a building block of eigensolvers, of other Krylov solvers
and of measurements), one solve (``solve_device``), and one solve for several
right-hand sides (``solve_batch_device``).  A case is one such call.

An operator that is asked for in a precision below FP64 returns numbers of
that precision in an FP64 buffer (every value is an FP32 number); the program
then keeps them as FP32, which loses nothing.  Solves with a fixed number of
iterations are the relaxed solves of all-mode averaging; their solutions are
kept in FP32 as well.  Solves to a residual return FP64.
"""
import math

import torch

import paper_2104_05615_amd as mspcg

# Moebius parameters of every workload of this repository
B, C, M5 = 1.5, 0.5, 1.8


def _case(name, kind, dims, Ls, **kw):
    c = {"name": name, "kind": kind, "X": dims[0], "Y": dims[1], "Z": dims[2], "T": dims[3], "Ls": Ls,
         "op": "", "prec": "fp32", "noalloc": False, "sub": "", "k": 0, "outer": "fp32", "inner": "fp16",
         "mf": 0.01, "eps": 0.5, "tol": 1e-10, "maxiter": 10000, "precond": True, "nrhs": 1}
    c.update(kw)
    return c


def _sub(s):
    return "x".join(str(v) for v in s)


def listed():
    return [
        # the smallest call: one hop on a test-sized lattice, all latency
        _case("dslash fp32 4^3x8 x8", "apply", (4, 4, 4, 8), 8, op="dslash_eo"),
        # an FP64 operator inside a tight loop on a small lattice, the entry point that allocates nothing
        _case("A fp64 8^4 x8 noalloc", "apply", (8, 8, 8, 8), 8, op="A", prec="fp64", noalloc=True, eps=0.3, mf=0.1),
        # ragged extents and an Ls that is no multiple of 4
        _case("Ddag fp32 6x10x14x18 x10", "apply", (6, 10, 14, 18), 10, op="Ddag"),
        # the normal operator of the outer solver at the ordinary volume
        _case("A fp32 16^3x32 x12", "apply", (16, 16, 16, 32), 12, op="A"),
        # the FP64 operator of residuals and source preparation at a serving volume
        _case("D fp64 24^3x48 x16", "apply", (24, 24, 24, 48), 16, op="D", prec="fp64", mf=0.001),
        # the subdomain operator in BF16, ragged tiling and Ls
        _case("A_sub bf16 12x8x20x24 x6", "apply", (12, 8, 20, 24), 6, op="A_sub", prec="bf16", sub=_sub((4, 4, 10, 8))),
        # the preconditioner in 8-bit storage on the multi-source workload's lattice
        _case("precond int8 16^4 x16", "apply", (16, 16, 16, 16), 16, op="precond", prec="int8", sub=_sub((4, 4, 4, 4)),
              k=6, mf=0.005),
        # the preconditioner at the ordinary volume
        _case("precond fp16 16^3x32 x12", "apply", (16, 16, 16, 32), 12, op="precond", prec="fp16",
              sub=_sub((4, 4, 4, 8)), k=6),
        # the outer operator and the preconditioner at the production shape
        _case("A fp32 32^3x64 x12", "apply", (32, 32, 32, 64), 12, op="A", eps=0.6, mf=0.00078),
        _case("precond fp16 32^3x64 x12", "apply", (32, 32, 32, 64), 12, op="precond", prec="fp16",
              sub=_sub((8, 8, 8, 16)), k=3, eps=0.6, mf=0.00078),
        # a whole mixed-precision MSPCG solve of the smallest serving volume, to the default residual
        _case("solve mixed 8^4 x8", "solve", (8, 8, 8, 8), 8, sub=_sub((4, 4, 4, 4)), k=5, eps=0.3, mf=0.1),
        # relaxed solves of twelve sources on one gauge field
        _case("batch 12 rhs 16^4 x16", "batch", (16, 16, 16, 16), 16, sub=_sub((4, 4, 4, 4)), k=6, mf=0.005, nrhs=12,
              maxiter=6),
    ]


def _even(rng, lo, hi):
    """An even number in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, 2 * int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 2))))


def _tiling(rng, dims):
    """Even divisors of the extents with the 4 sites outside that a partitioned direction needs."""
    out = []
    for d in dims:
        ok = [s for s in range(4, d + 1, 2) if d % s == 0 and (s == d or d - s >= 4)]
        small = [s for s in ok if s <= 10 and s < d]
        out.append(rng.choice(small or ok))
    return out


def draw(rng):
    kind = rng.choice(["apply"] * 7 + ["solve"] * 2 + ["batch"])
    Ls = rng.choice([4, 6, 8, 8, 10, 12, 12, 12, 16, 16])
    mf, eps = rng.choice([0.1, 0.01, 0.001]), rng.choice([0.3, 0.5, 0.6])
    if kind == "solve":
        dims = [_even(rng, 8, 12) for _ in range(3)] + [_even(rng, 8, 16)]
        pre = rng.random() < 0.6
        # plain CG, or MSPCG; FP64 throughout, or mixed
        fp64 = rng.random() < 0.3
        return _case("", "solve", dims, Ls, sub=_sub(_tiling(rng, dims)) if pre else "", k=rng.choice([3, 4, 5, 6]),
                     outer="fp64" if fp64 else "fp32", inner="fp64" if fp64 else rng.choice(["fp16", "int8", "bf16"]),
                     precond=pre, mf=0.1, eps=eps)
    if kind == "batch":
        dims = [_even(rng, 8, 16) for _ in range(4)]
        return _case("", "batch", dims, Ls, sub=_sub(_tiling(rng, dims)), k=rng.choice([3, 6]), mf=mf, eps=eps,
                     nrhs=rng.choice([2, 3, 5, 8, 12]), maxiter=rng.randint(2, 6))
    # volumes between the smallest and the largest listed ones
    while True:
        dims = [_even(rng, 4, 32) for _ in range(3)] + [_even(rng, 8, 64)]
        n = dims[0] * dims[1] * dims[2] * dims[3] * Ls
        if n <= 32 ** 3 * 64 * 12 // 2:
            break
    op = rng.choice(["dslash_eo", "dslash_dag_oe", "D", "Ddag", "A", "A", "A_sub", "precond", "precond"])
    if op in ("A_sub", "precond"):
        # room for subdomains; the regions around small ones are several times the lattice
        dims = [max(8, d) for d in dims]
        while dims[0] * dims[1] * dims[2] * dims[3] * Ls > 32 ** 3 * 64 * 12 // 4:
            m = max(range(4), key=lambda i: dims[i])
            dims[m] -= 2
        return _case("", "apply", dims, Ls, op=op, prec=rng.choice(["fp16", "fp16", "int8", "bf16", "fp32"]),
                     sub=_sub(_tiling(rng, dims)), k=rng.choice([3, 4]), mf=mf, eps=eps)
    return _case("", "apply", dims, Ls, op=op, prec=rng.choice(["fp32", "fp32", "fp64"]), mf=mf, eps=eps)


# ---------------------------------------------------------------- inputs

def _mm(a, b):
    """Products of 3 x 3 matrices held as nested lists of tensors."""
    return [[a[i][0] * b[0][j] + a[i][1] * b[1][j] + a[i][2] * b[2][j] for j in range(3)] for i in range(3)]


def _links(case, gen):
    """Random SU(3) links U = exp(i eps H), H the traceless Hermitian part of a
    complex Gaussian matrix: [T][Z][Y][X][4][3][3] complex128 on the GPU."""
    n = case["X"] * case["Y"] * case["Z"] * case["T"] * 4
    g = torch.randn((3, 3, 2, n), generator=gen, device="cuda", dtype=torch.float64)
    G = torch.complex(g[:, :, 0], g[:, :, 1])
    del g
    H = 0.5 * (G + G.transpose(0, 1).conj())
    tr = (H[0, 0] + H[1, 1] + H[2, 2]).real / 3.0
    for i in range(3):
        H[i, i] -= tr
    H *= 1j * case["eps"] / 32.0
    A = [[H[i, j].clone() for j in range(3)] for i in range(3)]
    del G, H
    # exp(A) = 1 + A/1 (1 + A/2 (1 + ... A/12)), then five squarings
    P = [[A[i][j] / 12.0 + float(i == j) for j in range(3)] for i in range(3)]
    for m in range(11, 0, -1):
        P = _mm(A, P)
        P = [[P[i][j] / m + float(i == j) for j in range(3)] for i in range(3)]
    for _ in range(5):
        P = _mm(P, P)
    U = torch.empty((n, 3, 3), device="cuda", dtype=torch.complex128)
    for i in range(3):
        for j in range(3):
            U[:, i, j] = P[i][j]
    return U.reshape(case["T"], case["Z"], case["Y"], case["X"], 4, 3, 3)


def _dims(case):
    return case["X"], case["Y"], case["Z"], case["T"]


def _source(case, gen):
    vh = case["X"] * case["Y"] * case["Z"] * case["T"] // 2
    shape = (case["nrhs"], case["Ls"], vh, 4, 3, 2)
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    U = _links(case, gen)
    return U, _source(case, gen)


_stream = None


def _program_stream():
    """The stream the program enqueues its work on (the library takes NULL as its own stream)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def prepare(case, seed):
    st = _program_stream()
    with torch.cuda.stream(st):
        U, src = _inputs(case, seed)
        host = U.cpu().numpy()
        del U
        out = torch.empty_like(src)
    torch.cuda.synchronize()
    h = mspcg.MSPCG(_dims(case))
    h.load_gauge(host)
    h.set_mobius(case["Ls"], B, C, M5, case["mf"])
    if case["sub"]:
        h.set_subdomains([int(v) for v in case["sub"].split("x")])
    h.set_solver(tol=case["tol"], maxiter=case["maxiter"], inner_iters=max(1, case["k"]), inner_prec=case["inner"],
                 outer_prec=case["outer"], use_precond=case["precond"])
    return {"case": case, "h": h, "src": src, "out": out, "stream": st}


def run(state):
    case, h, src, out, st = state["case"], state["h"], state["src"], state["out"], state["stream"]
    with torch.cuda.stream(st):
        if case["kind"] == "apply":
            f = h.apply_device_noalloc if case["noalloc"] else h.apply_device
            f(case["op"], case["prec"], src.data_ptr(), out.data_ptr(), st.cuda_stream)
            return out if case["prec"] == "fp64" else out.float()
        if case["kind"] == "solve":
            h.solve_device(src.data_ptr(), out.data_ptr(), None, st.cuda_stream)
            return out
        h.solve_batch_device(case["nrhs"], src.data_ptr(), out.data_ptr(), None, st.cuda_stream)
        return out.float()


def work(case):
    """One pass: the source in, the result out, the links once, and the
    arithmetic of the operators (a hop is 1320 flops per 5D site; a
    fifth-dimension matrix 48 Ls)."""
    vh, Ls = case["X"] * case["Y"] * case["Z"] * case["T"] // 2, case["Ls"]
    size = {"fp64": 8, "fp32": 4, "bf16": 2, "fp16": 2, "int8": 2}[case["prec"] if case["kind"] == "apply" else "fp32"]
    links = 2 * vh * 4 * 18 * size
    fields = 2 * case["nrhs"] * Ls * vh * 24 * 8
    hop, mat = 1320.0 * Ls * vh, 48.0 * Ls * Ls * vh
    A = 4 * hop + 7 * mat
    if case["kind"] == "apply":
        f = {"dslash_eo": hop, "dslash_dag_oe": hop, "D": 2 * hop + 3 * mat, "Ddag": 2 * hop + 3 * mat, "A": A,
             "A_sub": A, "precond": case["k"] * A}[case["op"]]
        return {"bytes": links + fields, "flops": f}
    # a solve to a residual takes at least some tens of iterations
    its = case["maxiter"] if case["maxiter"] < 10000 else 30
    per = A + (case["k"] * A if case["precond"] else 0)
    return {"bytes": links + fields * its, "flops": its * per * case["nrhs"]}


# ---------------------------------------------------------------- the same in 64 bits
#
# Plain torch on whole arrays.  A field is [4 spins][3 colours][Ls][n][t][z][y][x]
# (both parities, n independent boxes), links are [mu][3][3][n][t][z][y][x].

# gamma_mu = [[0, G_mu], [G_mu^dag, 0]], G_k = -i sigma_k, G_t = 1: G_mu psi_down as
# (factor, spin) of the two upper spins, and G_mu^dag psi_up of the two lower ones
_UP = [[(-1j, 3), (-1j, 2)], [(-1, 3), (1, 2)], [(-1j, 2), (1j, 3)], [(1, 2), (1, 3)]]
_DN = [[(1j, 1), (1j, 0)], [(1, 1), (-1, 0)], [(1j, 0), (-1j, 1)], [(1, 0), (1, 1)]]


def _gamma(mu, p, sign):
    """(1 + sign gamma_mu) p"""
    rows = _UP[mu] + _DN[mu]
    return [p[s] + (sign * rows[s][0]) * p[rows[s][1]] for s in range(4)]


def _hop64(U, p, dagger):
    """D^w: sum_mu (1 - gamma) U(x) psi(x + mu) + (1 + gamma) U^dag(x - mu) psi(x - mu); adjoint: signs exchanged."""
    out = torch.zeros_like(p)
    for mu in range(4):
        ax = -1 - mu
        for fwd in (True, False):
            sign = (-1 if fwd else 1) * (-1 if dagger else 1)
            h = _gamma(mu, torch.roll(p, -1 if fwd else 1, dims=ax), sign)
            u = U[mu] if fwd else torch.roll(U[mu], 1, dims=ax)
            for s in range(4):
                for a in range(3):
                    for b in range(3):
                        w = u[a, b] if fwd else u[b, a].conj()
                        out[s, a] += w * h[s][b]
    return out


class _Op64:
    """D, D^dag and A of one parity, with the fifth-dimension matrices as dense Ls x Ls ones per chirality."""

    def __init__(self, case, U):
        Ls, mf = case["Ls"], case["mf"]
        self.U = U
        S = torch.zeros((Ls, Ls), dtype=torch.float64)
        for s in range(1, Ls):
            S[s, s - 1] = 1.0
        S[0, Ls - 1] = -mf
        one = torch.eye(Ls, dtype=torch.float64)
        m5 = (B * (4 - M5) + 1) * one + (C * (4 - M5) - 1) * S
        mphi = -0.5 * (B * one + C * S)
        inv = torch.linalg.inv(m5)
        dev = lambda m: (m.cuda(), m.t().contiguous().cuda())   # noqa: E731  the two chiralities
        self.m5, self.mphi, self.inv = dev(m5), dev(mphi), dev(inv)

    @staticmethod
    def mat(M, p, dagger=False):
        out = torch.empty_like(p)
        for s in range(4):
            m = M[(s >= 2) != dagger]
            for a in range(3):
                f = torch.view_as_real(p[s, a]).reshape(p.shape[2], -1)
                out[s, a] = torch.view_as_complex((m @ f).reshape(*p.shape[2:], 2))
        return out

    def hop(self, p, dagger=False):
        return _hop64(self.U, p, dagger)

    def D(self, p, keep=None):
        a = self.mat(self.inv, self.hop(self.mat(self.mphi, p)))
        return p - self.mat(self.inv, self.hop(self.mat(self.mphi, a)))

    def Ddag(self, p):
        a = self.mat(self.mphi, self.hop(self.mat(self.inv, p, True), True), True)
        return p - self.mat(self.mphi, self.hop(self.mat(self.inv, a, True), True), True)

    def A(self, p):
        return self.Ddag(self.D(p))


def _sites(case, parity):
    """x, y, z, t of the sites of one parity in the library's order (lex / 2)."""
    X, Y, Z, T = _dims(case)
    lex = 2 * torch.arange(X * Y * Z * T // 2, device="cuda")
    y, z, t = (lex // X) % Y, (lex // (X * Y)) % Z, lex // (X * Y * Z)
    return lex % X + ((y + z + t + parity) & 1), y, z, t


def _spread(case, v, parity):
    """[Ls][V/2][4][3][2] of one parity -> whole-lattice field, zero on the other."""
    X, Y, Z, T = _dims(case)
    x, y, z, t = _sites(case, parity)
    f = torch.zeros((4, 3, case["Ls"], 1, T, Z, Y, X), dtype=torch.complex128, device="cuda")
    f[:, :, :, 0, t, z, y, x] = torch.view_as_complex(v).permute(2, 3, 0, 1)
    return f


def _gather(case, f, parity):
    x, y, z, t = _sites(case, parity)
    return torch.view_as_real(f[:, :, :, 0, t, z, y, x].permute(2, 3, 0, 1).contiguous())


def _precond64(case, U, f, k):
    """k CG iterations from zero on R_s A R_s^T of every subdomain, or (k = 0) R_s A R_s^T itself.

    A subdomain with the two sites around it (in partitioned directions) as a
    periodic box: four hops from inside it and back never notice the wrap."""
    dims, sub = _dims(case), [int(v) for v in case["sub"].split("x")]
    pad = [0 if s == d else 2 for s, d in zip(sub, dims)]
    out = torch.zeros_like(f)
    corners = [(x, y, z, t) for t in range(0, dims[3], sub[3]) for z in range(0, dims[2], sub[2])
               for y in range(0, dims[1], sub[1]) for x in range(0, dims[0], sub[0])]
    box = math.prod(s + 2 * p for s, p in zip(sub, pad))
    group = max(1, min(len(corners), int(3e6 * 12 / case["Ls"]) // box))
    for g0 in range(0, len(corners), group):
        cs = corners[g0:g0 + group]
        idx = []
        for m in range(4):
            i = torch.tensor([[(c[m] + o) % dims[m] for o in range(-pad[m], sub[m] + pad[m])] for c in cs], device="cuda")
            shape = [len(cs), 1, 1, 1, 1]
            shape[4 - m] = i.shape[1]
            idx.append(i.reshape(shape))
        at = (idx[3], idx[2], idx[1], idx[0])
        op = _Op64(case, [U[m][:, :, 0][(slice(None), slice(None)) + at] for m in range(4)])
        inside = tuple(slice(pad[m], pad[m] + sub[m]) for m in (3, 2, 1, 0))
        mask = torch.zeros([len(cs)] + [sub[m] + 2 * pad[m] for m in (3, 2, 1, 0)], dtype=torch.float64, device="cuda")
        mask[(slice(None),) + inside] = 1.0
        r = f[:, :, :, 0][(slice(None),) * 3 + at] * mask
        As = lambda p: op.A(p) * mask   # noqa: E731
        if k == 0:
            z = As(r)
        else:
            dot = lambda a, b: (torch.view_as_real(a) * torch.view_as_real(b)).sum(dim=(0, 1, 2, 4, 5, 6, 7, 8))   # noqa: E731
            over = lambda a, b: torch.where(b > 0, a / torch.where(b > 0, b, torch.ones_like(b)), torch.zeros_like(b))   # noqa: E731
            wide = lambda a: a.reshape(-1, 1, 1, 1, 1)   # noqa: E731
            # the other parity is zero, so a box's sums are those of its even sites
            z, p, rho = torch.zeros_like(r), r.clone(), dot(r, r)
            for it in range(k):
                q = As(p)
                al = wide(over(rho, dot(p, q)))
                z += al * p
                if it + 1 < k:
                    r -= al * q
                    new = dot(r, r)
                    p = r + wide(over(new, rho)) * p
                    rho = new
        flat = tuple(i.expand(mask.shape)[(slice(None),) + inside] for i in at)
        out[:, :, :, 0, flat[0], flat[1], flat[2], flat[3]] = z[(slice(None),) * 4 + inside]
    return out


def exact(case, seed):
    if case["kind"] == "batch":
        return None   # the iterates of a relaxed solve depend on the storage of its preconditioner
    vol = case["X"] * case["Y"] * case["Z"] * case["T"]
    if case["kind"] == "solve" and vol * case["Ls"] > 16 ** 3 * 32 * 12:
        return None
    Uh, src = _inputs(case, seed)
    U = [Uh[..., mu, :, :].permute(4, 5, 0, 1, 2, 3).unsqueeze(2).contiguous() for mu in range(4)]
    del Uh
    src = src[0]
    if case["kind"] == "solve":
        # CG far past the residual the solve stops at
        op = _Op64(case, U)
        b = _spread(case, src, 0)
        x, r = torch.zeros_like(b), b.clone()
        p, rho = r.clone(), float(torch.view_as_real(r).square().sum())
        stop = rho * 1e-28
        for _ in range(4000):
            q = op.A(p)
            al = rho / float((torch.view_as_real(p) * torch.view_as_real(q)).sum())
            x += al * p
            r -= al * q
            new = float(torch.view_as_real(r).square().sum())
            if new < stop:
                break
            p = r + (new / rho) * p
            rho = new
        return _gather(case, x, 0).unsqueeze(0)
    op = case["op"]
    if op in ("A_sub", "precond"):
        f = _spread(case, src, 0)
        return _gather(case, _precond64(case, U, f, case["k"] if op == "precond" else 0), 0).unsqueeze(0)
    o = _Op64(case, U)
    if op == "dslash_eo":
        return _gather(case, o.hop(_spread(case, src, 1)), 0).unsqueeze(0)
    if op == "dslash_dag_oe":
        return _gather(case, o.hop(_spread(case, src, 0), True), 1).unsqueeze(0)
    f = _spread(case, src, 0)
    return _gather(case, {"D": o.D, "Ddag": o.Ddag, "A": o.A}[op](f), 0).unsqueeze(0)
