"""Workloads the library's speed is measured on: whole calls of its public entry points.

Every case is one call a program makes with its inputs resident on the GPU and a
Context it keeps (created by ``prepare``):

  density   P0 at a fixed chemical potential (``Context.fermi_recursion``)
  newton    canonical responses of order 0, 1 or 2 (``Context.mu_newton``)
  grad      forward and backward of the differentiable density matrix (``fermi_canonical``)
  batch     many uneven systems in one call (``Context.mu_newton_batched``)
  sparse    the thresholded block-sparse form (``Context.sparse_response``)
  basis     a response in a non-orthogonal basis (``Context.mu_newton_nonorthogonal``)

Hamiltonians are the package's tight-binding models (``workloads``), seeded;
perturbations are dipoles along the lattice axes.  beta and the recursion depth
follow the model: 10 and 20 for chains, 20 and 25 for cubic lattices, 40 and 30 for
banded matrices.  Sizes span those of the named workloads (128 to 4096 here; the banded
8192 one takes longer than a case may), ragged ones among them.
"""
import math

import numpy as np
import torch

import paper_1503_07037_amd as dm
import workloads
from paper_1503_07037_amd.autograd import fermi_canonical

# context options by name: the library's defaults (FP64 products, conjugate gradients), FP64 with the
# shared inverse, the benchmark's form (int8 slices), and the FP32 products of the batched and
# adjoint workloads
FORMS = {
    "default": dict(),
    "fp64": dict(prec="fp64", solver="hybrid"),
    "int8": dict(prec="int8x6", refine=2, solver="hybrid"),
    "fp32": dict(prec="fp32"),
}
BETA_N = {"chain": (10.0, 20), "dimer": (10.0, 22), "cubic": (20.0, 25), "banded": (40.0, 30)}


def listed():
    return [
        # the smallest call: P0 of a small molecule's Hamiltonian inside somebody else's loop
        dict(name="density_96", kind="density", form="default", model="chain", N=96),
        # the 128-site chain with its dipole response, orders 0 to 2, library defaults
        dict(name="chain_128", kind="newton", form="default", model="chain", N=128, order=2, dirs=1),
        # a canonical density matrix per molecular-dynamics step, ragged size, library defaults
        dict(name="density_701", kind="newton", form="default", model="banded", N=701, order=0, dirs=0),
        # polarisability tensor of a 10^3 lattice in FP64
        dict(name="lattice_1000_fp64", kind="newton", form="fp64", model="cubic", lx=10, ly=10, lz=10,
             order=1, dirs=3),
        # hyperpolarisability in FP64, the accuracy-matched form of the benchmark, ragged size
        dict(name="banded_2310_fp64", kind="newton", form="fp64", model="banded", N=2310, order=2, dirs=3),
        # the 16 x 16 x 8 lattice, one direction, in the benchmark's int8 form
        dict(name="cubic_2048_int8", kind="newton", form="int8", model="cubic", lx=16, ly=16, lz=8,
             order=2, dirs=1),
        # the benchmark's recipe (banded, three directions, orders 0 to 2) at half its size
        dict(name="banded_4096_int8", kind="newton", form="int8", model="banded", N=4096, order=2, dirs=3),
        # force-like training step: density matrix forward, gradient with respect to H0 backward
        dict(name="grad_1728_fp32", kind="grad", form="fp32", model="cubic", lx=12, ly=12, lz=12),
        # a batch of uneven lattices with three directions (the batched workload's recipe, fewer systems)
        dict(name="batch_8_fp32", kind="batch", form="fp32", count=8, lo=256, hi=1024, order=2, dirs=3),
        # many small molecules, one direction
        dict(name="batch_24_small", kind="batch", form="fp32", count=24, lo=40, hi=250, order=1, dirs=1),
        # linear-scaling form of a gapped chain
        dict(name="sparse_2048", kind="sparse", form="default", model="dimer", N=2048, order=2, dirs=1),
        # one response of a non-orthogonal (Gaussian-like) basis
        dict(name="basis_500", kind="basis", form="default", model="chain", N=500, order=1, dirs=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["density", "default", "fp64", "fp64", "int8", "int8", "grad", "batch", "small",
                       "sparse", "basis"])
    if kind == "density":
        return dict(kind="density", form="default", model=rng.choice(["chain", "banded"]), N=_log_int(rng, 50, 700))
    if kind == "default":
        return dict(kind="newton", form="default", model=rng.choice(["chain", "banded"]), N=_log_int(rng, 80, 900),
                    order=rng.choice([0, 1, 2]), dirs=1)
    if kind == "fp64":
        return dict(kind="newton", form="fp64", model="banded", N=_log_int(rng, 300, 2300), order=rng.choice([0, 1, 2]),
                    dirs=rng.choice([1, 2, 3]))
    if kind == "int8":
        return dict(kind="newton", form="int8", model="banded", N=_log_int(rng, 900, 4000), order=rng.choice([0, 1, 2]),
                    dirs=rng.choice([1, 2, 3]))
    if kind == "grad":
        e = [rng.randint(6, 12) for _ in range(3)]
        return dict(kind="grad", form="fp32", model="cubic", lx=e[0], ly=e[1], lz=e[2])
    if kind == "batch":
        return dict(kind="batch", form="fp32", count=rng.randint(3, 8), lo=150, hi=rng.randint(400, 1024),
                    order=rng.choice([1, 2]), dirs=rng.choice([1, 2, 3]))
    if kind == "small":
        return dict(kind="batch", form="fp32", count=rng.randint(8, 28), lo=30, hi=rng.randint(80, 250), order=1, dirs=1)
    if kind == "sparse":
        return dict(kind="sparse", form="default", model="dimer", N=_log_int(rng, 700, 3000), order=rng.choice([1, 2]),
                    dirs=1)
    return dict(kind="basis", form="default", model="chain", N=_log_int(rng, 150, 700), order=rng.choice([0, 1]), dirs=1)


# ------------------------------------------------------------------ inputs
def _gpu(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _grid(n):
    """(lx, ly, lz) of a grid that holds n points, near-cubic, z slowest."""
    ly = max(1, int(round(n ** (1.0 / 3.0))))
    lx = ly
    return lx, ly, -(-n // (lx * ly))


def _axes(n):
    """Centred coordinates of n points read off a near-cubic grid."""
    lx, ly, lz = _grid(n)
    i = np.arange(n)
    return [i % lx - lx / 2.0, i // lx % ly - ly / 2.0, i // (lx * ly) - lz / 2.0]


def _system(case, seed):
    """Host H0, the axes' coordinates, beta, n and Ne of a case with one system."""
    model = case["model"]
    beta, n = BETA_N[model]
    if model == "cubic":
        dims = case["lx"], case["ly"], case["lz"]
        h0 = workloads.cubic_lattice(*dims, seed)
        x = list(workloads.lattice_dipoles(*dims))
    else:
        N = case["N"]
        if model == "chain":
            h0 = workloads.chain_1d(N, seed)
            x = [np.arange(N) - N / 2.0]
        elif model == "dimer":
            h0 = workloads.dimer_chain(N, seed)
            x = [(np.arange(N) - N / 2.0) / N]
        else:
            h0 = workloads.banded(N, seed)
            x = _axes(N)
    return h0, x[:case.get("dirs", 0)], beta, n, float(h0.shape[0] // 2)


def _batch(case, seed):
    """Host systems of a batch: sizes of the case alone, Hamiltonians from the seed."""
    sizes = np.random.default_rng(case["count"] * 1000 + case["hi"])
    got = []
    for k in range(case["count"]):
        t = math.exp(sizes.uniform(math.log(case["lo"]), math.log(case["hi"])))
        e = max(2, int(round(t ** (1.0 / 3.0))))
        dims = (max(2, min(int(round(t / (e * e))), case["hi"] // (e * e))), e, e)
        h0 = workloads.cubic_lattice(*dims, 1000 * seed + k)
        x = list(workloads.lattice_dipoles(*dims))[:case["dirs"]]
        got.append((h0, x, float(sizes.uniform(5.0, 40.0)), h0.shape[0] / 2.0))
    return got


def _cotangent(n, seed):
    """A symmetric banded cotangent of P0, as a loss on local matrix elements gives it."""
    return workloads.banded(n, seed + 77, bandwidth=16, sigma=0.5, decay=4.0, diag=1.0)


def prepare(case, seed):
    opts = FORMS[case["form"]]
    kind = case["kind"]
    s = dict(case=case)
    if kind == "batch":
        sysm = _batch(case, seed)
        s["H0s"] = [_gpu(h) for h, _, _, _ in sysm]
        s["H1s"] = [[_gpu(np.diag(v)) for v in x] for _, x, _, _ in sysm]
        s["betas"], s["Nes"] = [b for _, _, b, _ in sysm], [e for _, _, _, e in sysm]
        s["ctx"] = dm.Context(max(h.shape[0] for h in s["H0s"]), dirs_max=case["dirs"], **opts)
        return s
    h0, x, beta, n, ne = _system(case, seed)
    N = h0.shape[0]
    s.update(H0=_gpu(h0), H1=[_gpu(np.diag(v)) for v in x], beta=beta, n=n, Ne=ne)
    if kind == "grad":
        s["A"] = _gpu(_cotangent(N, seed))
    if kind == "basis":
        s["Z"] = _gpu(workloads.inverse_factor(workloads.overlap(N, seed)))
    # the sparse form does not use the context's dense workspace
    s["ctx"] = dm.Context(128 if kind == "sparse" else N, dirs_max=case.get("dirs", 0), **opts)
    return s


# ------------------------------------------------------------------ the calls
MU_FIXED = 0.05


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "batch":
        P0, P1, P2, mus, _ = ctx.mu_newton_batched(s["H0s"], s["H1s"], s["betas"], s["Nes"], n=25, order=case["order"])
        return dict(P0=P0, P1=P1, P2=P2, mu=np.array(mus))
    if kind == "density":
        P0, _ = ctx.fermi_recursion(s["H0"], s["beta"], MU_FIXED, s["n"])
        return dict(P0=P0)
    if kind == "grad":
        H0 = s["H0"].detach().requires_grad_(True)
        P0 = fermi_canonical(H0, s["beta"], s["Ne"], s["n"], ctx)
        P0.backward(s["A"])
        return dict(P0=P0.detach(), G=H0.grad)
    if kind == "sparse":
        P0, P1, P2, mu, _ = ctx.sparse_response(s["H0"], s["H1"], beta=s["beta"], Ne=s["Ne"], n=s["n"],
                                                order=case["order"], tau=1e-8, count_thr=1e-5, blocks_per_row=64)
    elif kind == "basis":
        P0, P1, P2, mu, _ = ctx.mu_newton_nonorthogonal(s["H0"], s["Z"], s["H1"], beta=s["beta"], Ne=s["Ne"], n=s["n"],
                                                        order=case["order"])
    else:
        P0, P1, P2, mu, _ = ctx.mu_newton(s["H0"], s["H1"], beta=s["beta"], Ne=s["Ne"], n=s["n"], order=case["order"])
    return dict(P0=P0, P1=P1, P2=P2, mu=np.array(mu))


# ------------------------------------------------------------------ work
def _dense_work(N, n, order, d):
    """One pass of the recursion: per step two N^3 products for order 0 (the square and the solve, both
    symmetric: half of 2 N^3 each), three more per direction at order 1, five at order 2; every input and
    output matrix once."""
    prods = 1.0 + (3.0 * d if order >= 1 else 0.0) + (5.0 * d if order >= 2 else 0.0)
    mats = 2 + (2 * d if order >= 1 else 0) + (d if order >= 2 else 0)
    return 2.0 * N ** 3 * n * prods, 8.0 * N * N * mats


def work(case):
    kind, order, d = case["kind"], case.get("order", 0), case.get("dirs", 0)
    if kind == "batch":
        both = [_dense_work(h.shape[0], 25, order, d) for h, _, _, _ in _batch(case, 0)]
        return dict(flops=sum(f for f, _ in both), bytes=sum(b for _, b in both))
    N = case["N"] if "N" in case else case["lx"] * case["ly"] * case["lz"]
    n = BETA_N[case["model"]][1]
    if kind == "grad":
        # forward and its reverse: per step one solve and two products for the cotangent
        f, b = _dense_work(N, n, 0, 0)
        return dict(flops=f + 2.0 * N ** 3 * n * 3.0, bytes=2.0 * b)
    flops, nbytes = _dense_work(N, n, order, d)
    if kind == "sparse":
        # about eleven blocks of 32 per block row meet eleven each; dense inputs and outputs
        flops *= 11.0 * 11.0 * 32.0 ** 2 / float(N) ** 2
    if kind == "basis":
        m = 1 + (d if order >= 1 else 0)
        flops += 2 * m * 2 * 2.0 * N ** 3
        nbytes += 8.0 * N * N
    return dict(flops=flops, bytes=nbytes)


# ------------------------------------------------------------------ the same in 64 bits, plain torch
def _inverse(S0):
    """(I + 4 S0)^-1 for S0 with eigenvalues in [0, 1/4]: Newton-Schulz from its best linear start."""
    eye = torch.eye(S0.shape[0], dtype=S0.dtype, device=S0.device)
    Tm = eye + 4.0 * S0
    Z = (24.0 * eye - 8.0 * Tm) / 17.0
    for _ in range(4):
        Z = 2.0 * Z - Z @ (Tm @ Z)
        Z = 0.5 * (Z + Z.T)
    return Z


def _expand(H0, E1, E2, beta, n, mu0):
    """n steps of D <- 2 D (I + 4 D^2)^-1 for H0 - mu0 I + lambda E1 + lambda^2 E2, by powers of
    lambda: P0, the list of P1, the list of P2 (E2: a matrix per direction, or nothing)."""
    eye = torch.eye(H0.shape[0], dtype=H0.dtype, device=H0.device)
    c = math.ldexp(beta, -(n + 2))
    D0, D1, D2 = c * (H0 - mu0 * eye), [c * e for e in E1], [c * e for e in E2]
    sym = lambda a: 0.5 * (a + a.T)
    for _ in range(n):
        S0 = D0 @ D0
        Z = _inverse(sym(S0))
        Y0 = sym(2.0 * (D0 @ Z))
        Y1, Y2 = [], []
        for z in range(len(D1)):
            S1 = D0 @ D1[z]
            S1 = S1 + S1.T
            Y1.append(sym(Z @ (2.0 * D1[z] - 4.0 * (S1 @ Y0))))
            if D2:
                S2 = D0 @ D2[z]
                S2 = S2 + S2.T + D1[z] @ D1[z]
                Y2.append(sym(Z @ (2.0 * D2[z] - 4.0 * (S1 @ Y1[z]) - 4.0 * (S2 @ Y0))))
        D0, D1, D2 = Y0, Y1, Y2
    return 0.5 * eye - D0, [-a for a in D1], [-a for a in D2]


def _canonical(H0, H1, beta, n, ne, order):
    """Tr P0 = Ne by a safeguarded Newton iteration, then Tr P1 = Tr P2 = 0 (affine in mu1, mu2)."""
    N = H0.shape[0]
    eye = torch.eye(N, dtype=H0.dtype, device=H0.device)
    off = (H0.abs().sum(1) - H0.diagonal().abs())
    lo, hi = float((H0.diagonal() - off).min()), float((H0.diagonal() + off).max())
    mu = float(H0.diagonal().sum()) / N
    best, found = math.inf, mu
    for _ in range(60):
        P0, _, _ = _expand(H0, [], [], beta, n, mu)
        e = float(P0.trace()) - ne
        if abs(e) < best:
            best, found = abs(e), mu
        elif best < 1e-9 * N:
            break
        if abs(e) < 1e-13 * N:
            break
        if e < 0.0:
            lo = max(lo, mu)
        else:
            hi = min(hi, mu)
        slope = beta * (float(P0.trace()) - float((P0 * P0).sum()))
        step = mu - e / slope if slope > 0.0 else math.nan
        mu = step if lo < step < hi else 0.5 * (lo + hi)
    mu, jet = found, [found]
    if order == 0:
        return _expand(H0, [], [], beta, n, mu) + (jet,)
    P0, P1, _ = _expand(H0, list(H1) + [eye], [], beta, n, mu)
    J = P1.pop()
    mu1 = [float(p.trace()) / float(J.trace()) for p in P1]
    P1 = [p - m * J for p, m in zip(P1, mu1)]
    jet = jet + mu1
    if order == 1:
        return P0, P1, [], jet
    _, _, P2 = _expand(H0, [h - m * eye for h, m in zip(H1, mu1)], [0.0 * H0 for _ in H1], beta, n, mu)
    mu2 = [float(p.trace()) / float(J.trace()) for p in P2]
    return P0, P1, [p - m * J for p, m in zip(P2, mu2)], jet + mu2


def exact(case, seed):
    kind, order = case["kind"], case.get("order", 0)
    if kind == "batch":
        all_ = []
        for h0, x, beta, ne in _batch(case, seed):
            P0, P1, P2, jet = _canonical(_gpu(h0), [_gpu(np.diag(v)) for v in x], beta, 25, ne, order)
            jet = jet + [0.0] * (1 + 2 * case["dirs"] - len(jet))
            all_.append((P0, P1, P2, jet))
        return dict(P0=[a[0] for a in all_], P1=[a[1] for a in all_],
                    P2=[a[2] for a in all_] if order >= 2 else [], mu=np.array([a[3] for a in all_]))
    h0, x, beta, n, ne = _system(case, seed)
    H0, H1 = _gpu(h0), [_gpu(np.diag(v)) for v in x]
    if kind == "density":
        return dict(P0=_expand(H0, [], [], beta, n, MU_FIXED)[0])
    if kind == "grad":
        # the canonical map is self-adjoint: its gradient is the first-order response to the cotangent
        P0, P1, _, _ = _canonical(H0, [_gpu(_cotangent(H0.shape[0], seed))], beta, n, ne, 1)
        return dict(P0=P0, G=P1[0])
    if kind == "basis":
        Z = _gpu(workloads.inverse_factor(workloads.overlap(H0.shape[0], seed)))
        P0, P1, P2, jet = _canonical(Z.T @ H0 @ Z, [Z.T @ h @ Z for h in H1], beta, n, ne, order)
        back = lambda p: Z @ p @ Z.T
        return dict(P0=back(P0), P1=[back(p) for p in P1], P2=[back(p) for p in P2], mu=np.array(jet))
    P0, P1, P2, jet = _canonical(H0, H1, beta, n, ne, order)
    return dict(P0=P0, P1=P1, P2=P2, mu=np.array(jet))
