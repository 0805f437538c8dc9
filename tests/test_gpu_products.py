"""GPU tests of the product kernels at the sizes where their tiling can go wrong.

FP64 products go through dmpt_congruence (two full products) against numpy, and
through the fixed-mu recursion with the shared inverse (symmetric products) against
the oracle: sizes on both sides of the 16-wide k chunks, the 32- and 64-wide tiles
(odd and even tile counts), the padding granule and the changes of tile edge.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def dm():
    import paper_1503_07037_amd as m
    m.load()
    return m


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_dev())


@pytest.mark.parametrize("n_max,sizes", [(700, (1, 15, 16, 17, 32, 33, 127, 128, 129, 500, 512, 513, 640, 700)),
                                         (1400, (1025, 1400, 65)), (4100, (4100, 3969, 130))])
def test_fp64_products_match_numpy(dm, n_max, sizes):
    """Z^T A Z by two full products; one context for falling and rising sizes, so stale padding
    would show.  Each entry is within the bound of two length-N FP64 sums, 4 N eps times the same
    sums of magnitudes."""
    rng = np.random.default_rng(5)
    with dm.Context(n_max, dirs_max=1, prec="fp64") as ctx:
        for N in sizes:
            print(f"case fp64 products N={N}", flush=True)
            Z = rng.standard_normal((N, N))
            A = rng.standard_normal((N, N))
            A = 0.5 * (A + A.T)
            for mode, L, R in ((0, Z.T, Z), (1, Z, Z.T)):
                B = ctx.congruence(T(Z), T(A), mode).cpu().numpy()
                ref = L @ A @ R
                bound = 4 * N * np.finfo(float).eps * (np.abs(L) @ np.abs(A) @ np.abs(R))
                assert (np.abs(B - ref) <= bound + 1e-300).all()


@pytest.mark.parametrize("n_max,sizes", [(700, (2, 31, 64, 97, 129, 384, 449, 513, 577, 640, 700)),
                                         (1400, (1400, 1153, 96))])
def test_fp64_symmetric_products_match_the_oracle(dm, n_max, sizes):
    """P0 at fixed mu with the shared inverse (every product symmetric; odd and even tile counts)."""
    beta, n, mu = 10.0, 20, 0.05
    with dm.Context(n_max, dirs_max=0, prec="fp64", solver="hybrid") as ctx:
        for N in sizes:
            print(f"case fp64 symmetric products N={N}", flush=True)
            h0 = workloads.chain_1d(N, 21)
            P0, _ = ctx.fermi_recursion(T(h0), beta, mu, n)
            p = P0.cpu().numpy()
            assert np.array_equal(p, p.T)
            assert np.abs(p - oracle.density(h0, beta, n, mu)).max() < 1e-12


@pytest.mark.parametrize("n_max,sizes", [(700, (2, 31, 33, 128, 129, 384, 385, 449, 577, 640, 700)), (1400, (1400, 96))])
def test_fp32_small_tiles_match_the_oracle(dm, n_max, sizes):
    """P0 at fixed mu with the default FP32 tiles, at the FP32 engine's accuracy (as in the parity tests)."""
    beta, n, mu = 10.0, 20, 0.05
    with dm.Context(n_max, dirs_max=0, prec="fp32") as ctx:
        for N in sizes:
            print(f"case fp32 products N={N}", flush=True)
            h0 = workloads.chain_1d(N, 22)
            p = ctx.fermi_recursion(T(h0), beta, mu, n)[0].cpu().numpy()
            assert np.array_equal(p, p.T)
            assert np.abs(p - oracle.density(h0, beta, n, mu)).max() < 1e-6


@pytest.mark.parametrize("prec,N", [("fp64", 90), ("fp64", 513), ("fp32", 300)])
def test_solves_that_run_ahead_of_the_host(dm, prec, N):
    """The conjugate-gradient solves queue iterations before the host knows that they are needed;
    with the product timing on they wait for every iteration instead.  Both give the same bits and
    statistics, and a solve that ends at max_cg is reported either way."""
    print(f"case solves {prec} N={N}", flush=True)
    h0, h1 = workloads.chain_1d(N, 3), [np.diag(np.linspace(-1.0, 1.0, N))]
    out = []
    with dm.Context(N, dirs_max=1, prec=prec) as ctx:
        for timed in (False, True):
            ctx.profile(timed)
            P0, P1, P2, mu, st = ctx.mu_newton(T(h0), [T(h) for h in h1], beta=10.0, Ne=N // 2, n=20, order=2)
            ctx.profile(False)
            out.append(([P0.cpu().numpy(), P1[0].cpu().numpy(), P2[0].cpu().numpy()], mu, st))
    (a, mu_a, sa), (b, mu_b, sb) = out
    assert all(np.array_equal(x, y) for x, y in zip(a, b)) and mu_a == mu_b
    for key in ("cg_iters_total", "cg_iters_max", "newton_iters"):
        assert sa[key] == sb[key]
    assert abs(sa["mfma_flops"] - sb["mfma_flops"]) <= 1e-12 * sb["mfma_flops"]
    for timed in (False, True):
        with dm.Context(N, dirs_max=1, prec=prec, max_cg=2) as ctx:
            ctx.profile(timed)
            with pytest.raises(dm.DMPTError):
                ctx.mu_newton(T(h0), [T(h) for h in h1], beta=10.0, Ne=N // 2, n=20, order=1)


@pytest.mark.parametrize("prec", ["int8x13", "int8x6"])
def test_int8_zero_digit_blocks(dm, monkeypatch, prec):
    """The int8 kernels (variants 0, 1) leave out the products of digit blocks that are zero; the variants
    with LDS DMA copies and the same wave tiles (2, 3) compute them all.  The digit sums are exact
    integers, so with whole diagonal tiles the results agree bit for bit: a scalar H0 (every iterate a multiple of I), narrow bands (whole
    stages without a product), entries spread over the digits' range, dense matrices, ragged sizes."""
    rng = np.random.default_rng(9)
    beta, n, mu = 8.0, 12, 0.07
    monkeypatch.setenv("DMPT_DIAG_SPLIT", "0")
    decay = np.exp(-0.05 * np.abs(np.subtract.outer(np.arange(1100), np.arange(1100))))
    dense = rng.standard_normal((1100, 1100))
    cases = [("scalar", 0.3 * np.eye(640)), ("chain", workloads.chain_1d(1000, 3)),
             ("decaying", (0.5 * (dense + dense.T)) * decay),
             ("dense", 0.02 * (dense + dense.T)[:300, :300]), ("tiny", 0.3 * np.ones((1, 1)))]
    for solver in ("ns", "cg"):
        for name, h0 in cases:
            N = h0.shape[0]
            print(f"case int8 zero blocks {prec} {solver} {name} N={N}", flush=True)
            out = []
            for v in (0, 1, 2, 3):
                with dm.Context(N, dirs_max=0, prec=prec, solver=solver, tol_cg=1e-6) as ctx:
                    ctx.set_variant(N, v)
                    out.append(ctx.fermi_recursion(T(h0), beta, mu, n)[0].cpu().numpy())
            assert np.array_equal(out[0], out[2]) and np.array_equal(out[1], out[3]), name


@pytest.mark.parametrize("solver", ["ns", "cg"])
def test_int8_slices_of_earlier_calls(dm, solver):
    """The slicing writes no zeros over zeros: after calls with denser, emptier, smaller and larger
    matrices a context gives bit for bit what a fresh one gives."""
    rng = np.random.default_rng(4)
    a = 0.02 * rng.standard_normal((640, 640))
    dense, chain, eye = a + a.T, workloads.chain_1d(640, 3), 0.3 * np.eye(640)
    mats = [dense, eye, chain, dense[:130, :130], chain, eye[:400, :400], dense[:400, :400], eye]
    opts = dict(dirs_max=0, prec="int8x13", solver=solver, tol_cg=1e-6)

    def solve(ctx, h0):
        return ctx.fermi_recursion(T(h0), 8.0, 0.07, 12)[0].cpu().numpy()

    with dm.Context(640, **opts) as used:
        for k, h0 in enumerate(mats):
            print(f"case int8 slices of earlier calls {solver} {k} N={h0.shape[0]}", flush=True)
            with dm.Context(640, **opts) as fresh:
                assert np.array_equal(solve(used, h0), solve(fresh, h0)), k


@pytest.mark.parametrize("N", [96, 200, 384, 500, 700, 1000, 1400])
def test_fp64_bits_do_not_depend_on_the_company(dm, N):
    """A direction gives the same bits alone and beside others, and a system of a batch the same
    whether products are launched per bucket or for all buckets together: the k groups a product's
    sums are split into follow from its size, not from the number of blocks of the launch."""
    print(f"case fp64 bits N={N}", flush=True)
    rng = np.random.default_rng(N)
    H0 = T(workloads.banded(N, 5))
    H1 = [T(np.diag(rng.standard_normal(N))) for _ in range(3)]
    with dm.Context(N, dirs_max=3, prec="fp64") as ctx:
        got = [ctx.response(H0, H1[:d], beta=10.0, n=20, order=1, mu=[0.05] + [0.0] * d) for d in (1, 2, 3)]
        for r in got[1:]:
            assert torch.equal(r[0], got[0][0]) and torch.equal(r[1][0], got[0][1][0])
    small = [64, N // 2, N]
    H0s = [H0] + [T(workloads.banded(e, 9 + i)) for i, e in enumerate(small)]
    H1s = [[H1[0]]] + [[T(np.diag(np.linspace(-1.0, 1.0, e)))] for e in small]
    out = []
    for count, grouped in ((1, 1), (4, 1), (4, 0)):
        with dm.Context(N, dirs_max=1, prec="fp64", grouped=grouped) as ctx:
            P0, P1, _, _, _ = ctx.mu_newton_batched(H0s[:count], H1s[:count], [10.0] * count,
                                                    [h.shape[0] / 2.0 for h in H0s[:count]], n=20, order=1)
            out.append((P0[0], P1[0][0]))
    for p0, p1 in out[1:]:
        assert torch.equal(p0, out[0][0]) and torch.equal(p1, out[0][1])
