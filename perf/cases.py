"""The workloads this framework is timed on, through its public entry points.

A case is one call that a user's program makes again and again: the action
exp(-i t H) psi of one instance (the plain call, from (h, J) or from a stored
diagonal, complex64 or complex128, Chebyshev or CF coefficients), a
polynomial of H, a time-dependent anneal, a batch of independent instances, or
the energy of a piecewise-constant anneal with its gradient.  Instances are
Sherrington-Kirkpatrick spin glasses (J ~ N(0, 1/n), h ~ N(0, 1)), states are
|+> (where quantum walks and anneals start) or a product state (a later stage
of a program).  The program keeps its output and workspace between calls.
"""
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

import paper_2608_12058_amd as qw

DEV = "cuda"


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # one dense-checkable walk of 10 qubits in double precision (the repository's
        # configuration 1): the smallest call, all latency
        dict(name="walk_n10_c128", kind="action", n=10, prec=128, gamma=1.0, t=1.0, tol=1e-12, method="cheb",
             source="tables", state="plus"),
        # the largest size that one workgroup holds, a longer walk: parameter scans
        # over many small instances run calls like this one after another
        dict(name="walk_n13_c64", kind="action", n=13, prec=64, gamma=0.7, t=5.0, tol=2.0 ** -23, method="cheb",
             source="tables", state="plus"),
        # a mid-size study instance of odd size
        dict(name="walk_n17_c64", kind="action", n=17, prec=64, gamma=1.3, t=5.0, tol=2.0 ** -23, method="cheb",
             source="tables", state="product"),
        # a problem given by its energies (not an Ising model), 20 qubits
        dict(name="walk_n20_c64_diag", kind="action", n=20, prec=64, gamma=1.0, t=6.0, tol=2.0 ** -23,
             method="cheb", source="diag", state="product"),
        # double precision at 21 qubits: reference results of a study
        dict(name="walk_n21_c128", kind="action", n=21, prec=128, gamma=0.8, t=3.0, tol=1e-12, method="cheb",
             source="tables", state="product"),
        # the repository's configuration 2: 24 qubits, CF coefficients
        dict(name="walk_n24_c64_cf", kind="action", n=24, prec=64, gamma=0.8, t=10.0, tol=2.0 ** -23, method="cf",
             source="tables", state="plus"),
        # the benchmark's 28-qubit instance over one unit of time: the largest call
        dict(name="walk_n28_c64", kind="action", n=28, prec=64, gamma=1.0, t=1.0, tol=2.0 ** -23, method="cheb",
             source="tables", state="plus"),
        # a polynomial of degree 50 with monomial coefficients, 26 qubits (Horner)
        dict(name="poly_n26_c64_mono", kind="poly", n=26, prec=64, gamma=1.0, degree=50, basis="mono",
             state="product"),
        # double precision above the memory-side cache: a polynomial of degree 50, 25 qubits
        dict(name="poly_n25_c128_cheb", kind="poly", n=25, prec=128, gamma=1.0, degree=50, basis="cheb",
             state="product"),
        # a linear anneal: many short exponentials on tables prepared once
        dict(name="anneal_n18_c64", kind="anneal", n=18, prec=64, T=2.0, steps=64, tol=1e-5, state="plus"),
        # independent instances of uneven size in one call, as the benchmark's batch draws them
        dict(name="batch48_n12_20", kind="batch", count=48, n_lo=12, n_hi=20, t_hi=20.0, tol=1e-6),
        # the repository's configuration 4: energy and gradient of 16 segments at 20 qubits
        dict(name="grad_n20_s16", kind="grad", n=20, segments=16, ckpt=8),
    ]


def draw(rng):
    """One more case of the ranges above (n counts qubits, so sizes are spread over their logarithm)."""
    kind = rng.choice(["action"] * 6 + ["poly", "poly", "anneal", "batch", "grad"])
    prec = rng.choice([64, 64, 64, 128])
    state = rng.choice(["plus", "product"])
    if kind == "action":
        n = rng.randint(8, 27 if prec == 64 else 25)
        # longer evolutions at small sizes, as in use; up to about a hundred terms at the largest
        t_hi = 10.0 if n <= 22 else (4.0 if n <= 24 else 1.2)
        return dict(kind=kind, n=n, prec=prec, gamma=round(rng.uniform(0.2, 2.0), 3),
                    t=round(math.exp(rng.uniform(math.log(0.3), math.log(t_hi))), 3),
                    tol=rng.choice([2.0 ** -23, 1e-6]) if prec == 64 else rng.choice([1e-12, 1e-10]),
                    method=rng.choice(["cheb", "cheb", "cf"]) if prec == 64 else "cheb",
                    source=rng.choice(["tables", "tables", "diag"]), state=state)
    if kind == "poly":
        return dict(kind=kind, n=rng.randint(8, 26 if prec == 64 else 24), prec=prec,
                    gamma=round(rng.uniform(0.2, 2.0), 3), degree=rng.randint(5, 60),
                    basis=rng.choice(["cheb", "mono"]), state=state)
    if kind == "anneal":
        n = rng.randint(8, 22)
        return dict(kind=kind, n=n, prec=prec, T=round(rng.uniform(0.5, 2.0), 3), steps=rng.randint(10, 64),
                    tol=rng.choice([1e-4, 1e-5]), state="plus")
    if kind == "batch":
        lo = rng.randint(10, 14)
        return dict(kind=kind, count=rng.randint(8, 48), n_lo=lo, n_hi=rng.randint(lo + 2, 20),
                    t_hi=round(rng.uniform(5.0, 20.0), 2), tol=1e-6)
    return dict(kind="grad", n=rng.randint(12, 20), segments=rng.randint(4, 16), ckpt=rng.choice([0, 8, -1]))


# ------------------------------------------------------------------ the inputs

def sk_instance(n, rng):
    J = rng.standard_normal(n * (n - 1) // 2) / math.sqrt(n)
    h = rng.standard_normal(n)
    return h, J


def make_state(n, kind, rng, dtype):
    if kind == "plus":
        return torch.full((1 << n,), 2.0 ** (-n / 2), dtype=dtype, device=DEV)
    f = rng.standard_normal((n, 2)) + 1j * rng.standard_normal((n, 2))
    f /= np.linalg.norm(f, axis=1, keepdims=True)
    f = torch.as_tensor(f, device=DEV).to(dtype)
    psi = f[0].clone()
    for j in range(1, n):
        psi = torch.cat([psi * f[j, 0], psi * f[j, 1]])   # qubit j: the next index bit
    return psi.contiguous()


def spins(m):
    return 1.0 - 2.0 * ((torch.arange(1 << m, device=DEV)[:, None] >> torch.arange(m, device=DEV)) & 1).double()


def energies(n, h, J):
    """E(z) = sum_{j<k} J_jk s_j s_k + sum_j h_j s_j in 64 bits, s_j = 1 - 2 bit_j(z), from two halves of the bits."""
    Jm = torch.zeros(n, n, dtype=torch.float64)
    iu = torch.triu_indices(n, n, 1)
    Jm[iu[0], iu[1]] = torch.as_tensor(J, dtype=torch.float64)
    Jm, h = Jm.to(DEV), torch.as_tensor(h, dtype=torch.float64).to(DEV)
    lo = n // 2
    sl, sh = spins(lo), spins(n - lo)
    El = ((sl @ Jm[:lo, :lo]) * sl).sum(1) + sl @ h[:lo]
    Eh = ((sh @ Jm[lo:, lo:]) * sh).sum(1) + sh @ h[lo:]
    return (sh @ (sl @ Jm[:lo, lo:]).T + Eh[:, None] + El[None, :]).reshape(-1)


def batch_sizes(case):
    """Uneven sizes n ~ U{n_lo..n_hi}, a part of the case; the seed draws the instances."""
    rng = np.random.default_rng(case["count"])
    return [int(n) for n in rng.integers(case["n_lo"], case["n_hi"] + 1, size=case["count"])]


def inputs(case, seed):
    """What the seed gives: couplings and states (torch, numpy)."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":
        insts = []
        for n in batch_sizes(case):
            t, g = float(rng.uniform(0.1, case["t_hi"])), float(rng.uniform(0.2, 2.0))
            h, J = sk_instance(n, rng)
            insts.append(dict(n=n, gamma=g, t=t, tol=case["tol"], h=h, J=J))
        return dict(case=case, insts=insts)
    n = case["n"]
    h, J = sk_instance(n, rng)
    if case["kind"] == "grad":
        S = case["segments"]
        leaf = lambda x: torch.as_tensor(np.asarray(x, dtype=np.float32)).requires_grad_()  # noqa: E731
        return dict(case=case, gammas=leaf(np.linspace(2.0, 0.05, S)), ts=leaf(np.full(S, 0.5)), h=leaf(h),
                    J=leaf(J), psi=make_state(n, "plus", rng, torch.complex64))
    prec = case["prec"]
    st = dict(case=case, h=h, J=J, diag=None)
    st["psi"] = make_state(n, case["state"], rng, torch.complex64 if prec == 64 else torch.complex128)
    if case.get("source") == "diag":
        st["diag"] = energies(n, h, J).to(torch.float32 if prec == 64 else torch.float64)
    if case["kind"] == "poly":
        st["coef"] = rng.standard_normal(case["degree"] + 1)
    return st


def prepare(case, seed):
    st = inputs(case, seed)
    if case["kind"] == "batch":
        st["batch"] = qw.Batch(st["insts"])
        for i, ins in enumerate(st["insts"]):
            st["batch"].state(i).fill_(2.0 ** (-ins["n"] / 2))
        st["stream"] = torch.cuda.Stream()
        st["stream"].wait_stream(torch.cuda.current_stream())
    elif case["kind"] != "grad":
        st["out"] = torch.empty_like(st["psi"])
        st["ws"] = qw.Workspace.for_problem(case["n"], case["prec"])
    return st


# -------------------------------------------------------------------- the calls

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "action":
        src = dict(diag=st["diag"]) if st["diag"] is not None else dict(h=st["h"], J=st["J"])
        out, _ = qw.expm_action(st["psi"], case["gamma"], case["t"], tol=case["tol"], method=case["method"],
                                out=st["out"], workspace=st["ws"], **src)
        return out
    if kind == "poly":
        out, _ = qw.poly_action(st["psi"], st["coef"], case["gamma"], basis=case["basis"], h=st["h"], J=st["J"],
                                out=st["out"], workspace=st["ws"])
        return out
    if kind == "anneal":
        out, _, _ = qw.anneal_cfet4(st["psi"], st["h"], st["J"], [0.0, 1.0], [1.0, -1.0], case["T"],
                                    steps=case["steps"], tol=case["tol"], out=st["out"], workspace=st["ws"])
        return out
    if kind == "batch":
        qw.expm_action_batched(st["batch"], stream=st["stream"])   # returns when its stream is done
        return st["batch"].out_pool
    # one step of a schedule optimisation in single precision: the loss and its gradients
    p = [st["gammas"], st["ts"], st["h"], st["J"]]
    E = qw.anneal_energy(*p, st["psi"], ckpt_every=case["ckpt"])
    return (E.detach().float(), *torch.autograd.grad(E, p))


# ---------------------------------------------------------------- what it needs

def degree(n, gamma, t, tol):
    """About the Chebyshev degree: the spectral radius of these instances is close to n (1 + gamma)."""
    a = abs(t) * n * (1.0 + gamma)
    return a + math.log(1.0 / tol) ** (2.0 / 3.0) * max(a, 1.0) ** (1.0 / 3.0) + 4.0


def vector_work(n, prec, terms):
    """A term reads b_{k+1}, b_{k+2} and psi and writes b_k, once vectors outgrow the chip's
    registers and LDS (about 170 MB); below that the call reads psi and writes its result.
    Per amplitude and term: n complex sums, the diagonal, the update."""
    N = float(1 << n)
    size = 8 if prec == 64 else 16
    moved = 4 * size * terms if 3 * size * N > 170e6 else 2 * size
    return N * moved, N * terms * (2 * n + 14)


def work(case):
    kind = case["kind"]
    if kind == "action":
        b, f = vector_work(case["n"], case["prec"], degree(case["n"], case["gamma"], case["t"], case["tol"]))
    elif kind == "poly":
        b, f = vector_work(case["n"], case["prec"], case["degree"])
    elif kind == "anneal":
        # two exponentials a step, on half a step's worth of H each
        t = 0.5 * case["T"] / case["steps"]
        b, f = vector_work(case["n"], case["prec"], 2.0 * case["steps"] * degree(case["n"], 0.0, t, case["tol"]))
    elif kind == "batch":
        each = [vector_work(n, 64, degree(n, 1.1, 0.5 * case["t_hi"], case["tol"])) for n in batch_sizes(case)]
        b, f = sum(x for x, _ in each), sum(y for _, y in each)
    else:
        terms = sum(degree(case["n"], g, 0.5, 2.0 ** -23) for g in np.linspace(2.0, 0.05, case["segments"]))
        b, f = vector_work(case["n"], 64, terms)
        f *= 2.5   # forward, and an adjoint step of about one and a half terms' operations
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------- in 64 bits, plain

def flips(n):
    """x -> sum_j x[z xor 2^j]: two products with the sums of a half's bit flips, or bit by bit."""
    if n <= 22:
        lo = n // 2

        def sums(m):
            X = torch.zeros(1 << m, 1 << m, dtype=torch.complex128, device=DEV)
            z = torch.arange(1 << m, device=DEV)
            for j in range(m):
                X[z, z ^ (1 << j)] = 1.0
            return X

        Xl, Xh = sums(lo), sums(n - lo)

        def apply(x):
            m = x.reshape(1 << (n - lo), 1 << lo)
            return (Xh @ m + m @ Xl).reshape(-1)
    else:
        def apply(x):
            y = torch.zeros_like(x)
            for j in range(n):
                a, b = x.view(-1, 2, 1 << j), y.view(-1, 2, 1 << j)
                b[:, 0] += a[:, 1]
                b[:, 1] += a[:, 0]
            return y
    return apply


def cheb_coef(a, tol=1e-15):
    """c_k of exp(-i a x) = sum_k c_k T_k(x), by a discrete cosine transform."""
    M = 1 << (int(2 * abs(a) + 200).bit_length() + 1)
    c = np.fft.fft(np.exp(-1j * a * np.cos(2 * np.pi * np.arange(M) / M))) / M
    c = c[:M // 2] * 2.0
    c[0] /= 2.0
    big = np.nonzero(np.abs(c) > tol)[0]
    return c[:int(big[-1]) + 2]


def clenshaw(coef, apply_h, v):
    """sum_k coef_k T_k(H) v; the vectors are used up as they go."""
    b1, b2 = torch.zeros_like(v), torch.zeros_like(v)
    for k in range(len(coef) - 1, 0, -1):
        b = apply_h(b1)
        b.mul_(2.0).sub_(b2).add_(v, alpha=complex(coef[k]))
        b1, b2 = b, b1
    y = apply_h(b1)
    return y.sub_(b2).add_(v, alpha=complex(coef[0]))


def scaled(n, E, gamma):
    """((H - c) / r applied to a vector, c, r)."""
    lo, hi = float(E.min()), float(E.max())
    c, r = 0.5 * (lo + hi), 0.5 * (hi - lo) + n * abs(gamma)
    d, F = (E - c) / r, flips(n)

    def apply(x):
        y = F(x).mul_(gamma / r)
        for i in range(0, x.numel(), 1 << 24):   # in pieces: no third vector
            y[i:i + (1 << 24)] += d[i:i + (1 << 24)] * x[i:i + (1 << 24)]
        return y

    return apply, c, r


def exp_action(n, E, gamma, t, v):
    apply, c, r = scaled(n, E, gamma)
    y = clenshaw(cheb_coef(t * r), apply, v)
    return y.mul_(complex(math.cos(t * c), -math.sin(t * c)))


def exact(case, seed):
    kind, st = case["kind"], inputs(case, seed)
    if kind == "batch":
        out = []
        for ins in st["insts"]:
            n = ins["n"]
            v = torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex64, device=DEV).to(torch.complex128)
            out.append(exp_action(n, energies(n, ins["h"], ins["J"]), ins["gamma"], ins["t"], v))
        return torch.cat(out)
    if kind == "grad":
        return exact_grad(case, st)
    n = case["n"]
    E = st["diag"].double() if st["diag"] is not None else energies(n, st["h"], st["J"])
    v = st.pop("psi").to(torch.complex128)
    if kind == "action":
        return exp_action(n, E, case["gamma"], case["t"], v)
    if kind == "anneal":
        return exact_anneal(case, E, v)
    apply = scaled(n, E, case["gamma"])[0]
    if case["basis"] == "cheb":
        return clenshaw(list(st["coef"]) + [0.0], apply, v)
    y = v * complex(st["coef"][-1])
    for a in st["coef"][-2::-1]:
        y = apply(y).add_(v, alpha=complex(a))
    return y


def exact_anneal(case, E, v):
    """The stated integrator in 64 bits: on every step two exponentials of H at the Gauss nodes."""
    n, T = case["n"], case["T"]
    lo, hi, F = float(E.min()), float(E.max()), flips(n)
    r3, hs = math.sqrt(3.0), T / case["steps"]
    a1, a2 = 0.25 + r3 / 6, 0.25 - r3 / 6
    for q in range(case["steps"]):
        s1, s2 = (q + 0.5 - r3 / 6) / case["steps"], (q + 0.5 + r3 / 6) / case["steps"]
        for w1, w2 in ((a1, a2), (a2, a1)):
            al, be = w1 * s1 + w2 * s2, w1 * (1 - s1) + w2 * (1 - s2)
            c, r = 0.5 * al * (lo + hi), abs(al) * 0.5 * (hi - lo) + n * abs(be)
            d = (al * E - c) / r
            v = clenshaw(cheb_coef(hs * r), lambda x: F(x).mul_(be / r).add_(d * x), v)
            v = v.mul_(complex(math.cos(hs * c), -math.sin(hs * c)))
    return v


def exact_grad(case, st):
    """Energy and gradient by autograd through the 64-bit series."""
    n, S = case["n"], case["segments"]
    p = [st[k].detach().double().to(DEV).requires_grad_() for k in ("gammas", "ts", "h", "J")]
    gam, ts, h, J = p
    s = spins(n)
    iu = torch.triu_indices(n, n, 1, device=DEV)
    Jm = torch.zeros(n, n, dtype=torch.float64, device=DEV).index_put((iu[0], iu[1]), J)
    E = ((s @ Jm) * s).sum(1) + s @ h
    lo, hi = float(E.detach().min()), float(E.detach().max())
    c, half = 0.5 * (lo + hi), 0.5 * (hi - lo)
    F = flips(n)
    psi = st["psi"].to(torch.complex128)

    def segment(psi, g, t, E):
        r = half + n * abs(float(g.detach()))
        K = len(cheb_coef(float(t.detach()) * r)) + 1
        M = 4 * K
        x = torch.cos(2 * math.pi * torch.arange(M, device=DEV, dtype=torch.float64) / M)
        ck = torch.fft.fft(torch.exp(-1j * (t * r) * x)) / M * 2.0
        d = (E - c) / r
        b1 = b2 = torch.zeros_like(psi)
        for k in range(K, 0, -1):
            b1, b2 = 2.0 * (d * b1 + (g / r) * F(b1)) - b2 + ck[k] * psi, b1
        y = d * b1 + (g / r) * F(b1) - b2 + 0.5 * ck[0] * psi
        return y * torch.exp(-1j * t * c)

    for q in range(S):
        psi = checkpoint(segment, psi, gam[q], ts[q], E, use_reentrant=False)
    loss = (E * (psi.real ** 2 + psi.imag ** 2)).sum()
    return [loss.detach(), *torch.autograd.grad(loss, p)]
