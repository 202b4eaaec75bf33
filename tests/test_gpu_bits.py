"""A product, and so an instance, has the same bits whatever shares its launch: every tile
shape sums in the same order.  Checked product by product over the shapes, and for
instances alone and among enough others that their launches take other shapes."""
import numpy as np
import pytest

from paper_2601_04904_amd.synth import gen_problem

pytestmark = pytest.mark.gpu
FIELDS = ("diag", "upper", "lower", "arrow_right", "arrow_bottom", "tip")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


@pytest.mark.parametrize("k", [0, 1, 15, 16, 17, 63, 64, 65, 79, 128, 129, 200])
@pytest.mark.parametrize("m,n", [(1, 1), (16, 17), (15, 33), (1, 200), (100, 37), (129, 127)])
@pytest.mark.parametrize("mixed", [False, True])
def test_product_bits_in_every_shape(torch, m, n, k, mixed):
    """shape -1 is the 16 x 16 tiles of a small launch at these sizes."""
    from paper_2601_04904_amd.solver import diag_gemm
    rng = np.random.default_rng(m * 1000 + n * 50 + k)
    for opA in (0, 1):
        for opB in (0, 1):
            dA = torch.from_numpy(crand(rng, *((k, m) if opA else (m, k)))).cuda()
            dB = torch.from_numpy(crand(rng, *((n, k) if opB else (k, n)))).cuda()
            dC = torch.from_numpy(crand(rng, m, n)).cuda()
            for alpha, beta, Cin in ((1.0, 1.0, dC), (-1.0, 1.0, dC), (1.0, 0.0, None), (0.5 - 2.0j, 0.25 - 1.5j, dC)):
                out = [diag_gemm(alpha, dA, opA, dB, opB, beta=beta, Cin=Cin, mixed=mixed, shape=s)
                       for s in (-1, 0, 1, 2)]
                for s in (1, 2, 3):
                    assert torch.equal(out[0], out[s]), (opA, opB, alpha, s - 1)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("specs", [[(6, 128, 0, 1)] * 16, [(5, 64, 37, 1)] * 24,
                                   [(9, 100, 20, 2), (6, 200, 64, 1), (7, 48, 0, 3), (4, 256, 0, 1)] * 5,
                                   # inverses: 40 of 120 apart, 300 in the shape of 520
                                   [(2, 300, 0, 1), (2, 520, 0, 1)] + [(2, 120, 0, 1)] * 40])
def test_instance_alone_and_among_many(torch, specs, precision):
    from paper_2601_04904_amd import solver as S
    kw = dict(precision=S.BT_MIXED, tol=1.0) if precision == "mixed" else {}
    probs = [gen_problem(n, b, a, 0.3, 0.05, 7 * i + b) for i, (n, b, a, _) in enumerate(specs)]

    def solve(which):
        dA = [S.DeviceBlocks.from_host(probs[i][0]) for i in which]
        dB = [S.DeviceBlocks.from_host(probs[i][1]) for i in which]
        XR, XL = ([S.DeviceBlocks.empty(*specs[i][:3]) for i in which] for _ in range(2))
        bs = S.BatchSolver([dict(n=specs[i][0], b=specs[i][1], a=specs[i][2], partitions=specs[i][3], **kw)
                            for i in which])
        err, fb = bs.solve(dA, dB, XR, XL)
        bs.sync()
        bs.destroy()
        return XR, XL, list(err), list(fb)

    R, L, err, fb = solve(range(len(specs)))
    for i in (0, 1, 2, 3, len(specs) - 1):
        r, l, e, f = solve([i])
        assert e[0] == err[i] and f[0] == fb[i], i
        for name in FIELDS:
            assert torch.equal(getattr(r[0], name), getattr(R[i], name)), (i, name)
            assert torch.equal(getattr(l[0], name), getattr(L[i], name)), (i, name)


@pytest.mark.parametrize("n,b,a,P", [(12, 96, 40, 2), (17, 201, 33, 4)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves_under_every_table(torch, n, b, a, P, precision):
    """A solve with every launch in one shape of the table has the bits of the untuned one,
    and is the oracle's."""
    import oracle
    from paper_2601_04904_amd import solver as S
    from tests._util import rel_err
    A, B = gen_problem(n, b, a, 0.3, 0.05, 5)
    dA, dB = S.DeviceBlocks.from_host(A), S.DeviceBlocks.from_host(B)
    saved = S.tune_table()
    out = []
    try:
        for v in (-1, 0, 1, 2):
            S.set_tune_table([v] * len(saved))
            XR, XL = S.DeviceBlocks.empty(n, b, a), S.DeviceBlocks.empty(n, b, a)
            sol = S.Solver(n, b, a, partitions=P,
                           **(dict(precision=S.BT_MIXED, tol=1.0) if precision == "mixed" else {}))
            sol.solve(dA, dB, XR, XL)
            sol.sync()
            sol.destroy()
            out.append((XR, XL))
    finally:
        S.set_tune_table(saved)
    for x in out[1:]:
        for i in (0, 1):
            for name in FIELDS:
                assert torch.equal(getattr(x[i], name), getattr(out[0][i], name)), (i, name)
    for x, ref in zip(out[0], oracle.solve_dense(A, B)):
        assert rel_err(x.to_host(), ref) < (1e-4 if precision == "mixed" else 1e-11)
