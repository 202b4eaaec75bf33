"""The product and inverse kernels at the sizes where their shapes change.

Products: k around the 16-deep stage, sizes around the tiles, every operand
order with alpha = -1 (a change of the accumulators' sign) and a general alpha
(multiplied into an operand), and launches of more than 128 products.  Inverses: dimensions
around each kernel shape, with rows that force pivoting.  Tolerances: a product
of k terms in FP64 is within (k + 4) eps of sum |a||b|; an inverse with partial
pivoting is held to 50 eps sqrt(d) cond, as the other inverse tests.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


@pytest.mark.parametrize("k", [1, 4, 15, 16, 17, 31, 32, 33, 47, 49])
@pytest.mark.parametrize("m,n", [(1, 65), (63, 31), (64, 64), (66, 33)])
@pytest.mark.parametrize("alpha", [1.0, -1.0, 0.5 - 2.0j])
def test_product_stage_edges(torch, m, n, k, alpha):
    from paper_2601_04904_amd.solver import diag_gemm
    rng = np.random.default_rng(m * 1000 + n * 50 + k)
    for opA in (0, 1):
        for opB in (0, 1):
            A = crand(rng, *((k, m) if opA else (m, k)))
            B = crand(rng, *((n, k) if opB else (k, n)))
            C = crand(rng, m, n)
            a, b = (A.conj().T if opA else A), (B.conj().T if opB else B)
            ref = C + alpha * (a @ b)
            bound = (k + 4) * EPS * 4 * (np.abs(C) + abs(alpha) * (np.abs(a) @ np.abs(b)))
            dA, dB, dC = (torch.from_numpy(x).cuda() for x in (A, B, C))
            for shape in (0, 1, 2):
                out = diag_gemm(alpha, dA, opA, dB, opB, beta=1.0, Cin=dC, shape=shape).cpu().numpy()
                assert (np.abs(out - ref) <= bound).all(), (opA, opB, shape)


@pytest.mark.parametrize("k", [0, 1, 15, 16, 17, 63, 64, 65, 80, 129, 1024])
@pytest.mark.parametrize("m,n", [(1, 1), (16, 17), (15, 33), (1, 200), (144, 16), (129, 127)])
def test_small_launch_tiles(torch, m, n, k):
    """The shape that the default rule takes for one small product: 16 x 16 tiles
    shared by the waves of a workgroup."""
    from paper_2601_04904_amd.solver import diag_gemm
    rng = np.random.default_rng(m * 1000 + n * 50 + k)
    beta = 0.25 - 1.5j
    EPS32 = np.finfo(np.float32).eps
    for opA in (0, 1):
        for opB in (0, 1):
            for alpha in (1.0, -1.0, 0.5 - 2.0j):
                A = crand(rng, *((k, m) if opA else (m, k)))
                B = crand(rng, *((n, k) if opB else (k, n)))
                C = crand(rng, m, n)
                a, b = (A.conj().T if opA else A), (B.conj().T if opB else B)
                dA, dB, dC = (torch.from_numpy(x).cuda() for x in (A, B, C))
                for Cin in (None, dC):
                    c0 = 0.0 if Cin is None else beta * C
                    bound = (k + 4) * EPS * 4 * (np.abs(c0) + abs(alpha) * (np.abs(a) @ np.abs(b)))
                    out = diag_gemm(alpha, dA, opA, dB, opB, beta=beta, Cin=Cin).cpu().numpy()
                    assert (np.abs(out - (c0 + alpha * (a @ b))) <= bound).all(), (opA, opB, alpha, Cin is None)
                    # products in complex64, beta C in FP64
                    out = diag_gemm(alpha, dA, opA, dB, opB, beta=beta, Cin=Cin, mixed=True).cpu().numpy()
                    bound += (k + 4) * EPS32 * 4 * abs(alpha) * (np.abs(a) @ np.abs(b))
                    assert (np.abs(out - (c0 + alpha * (a @ b))) <= bound).all(), (opA, opB, alpha, Cin is None)


def test_more_products_than_one_search(torch):
    """130 instances: launches of more than 128 products and inverses."""
    import oracle
    from tests._util import rel_err
    from paper_2601_04904_amd import solver as S
    from paper_2601_04904_amd.synth import gen_problem
    probs = [gen_problem(3, 4 + i % 3, i % 2, 0.3, 0.05, 7 * i) for i in range(130)]
    dA = [S.DeviceBlocks.from_host(A) for A, _ in probs]
    dB = [S.DeviceBlocks.from_host(B) for _, B in probs]
    XR = [S.DeviceBlocks.empty(A.n, A.b, A.a) for A, _ in probs]
    XL = [S.DeviceBlocks.empty(A.n, A.b, A.a) for A, _ in probs]
    bs = S.BatchSolver([dict(n=A.n, b=A.b, a=A.a) for A, _ in probs])
    bs.solve(dA, dB, XR, XL)
    bs.sync()
    for i, (A, B) in enumerate(probs):
        R, L = oracle.solve_dense(A, B)
        assert rel_err(XR[i].to_host(), R) < 1e-11, i
        assert rel_err(XL[i].to_host(), L) < 1e-11, i
    bs.destroy()


@pytest.mark.parametrize("sizes", [(113, 300), (256, 513), (40, 100, 128, 257), (200, 112)])
def test_inverse_shapes_in_one_level(torch, sizes):
    """Instances whose inverses have different kernel shapes, levelled together."""
    import oracle
    from tests._util import rel_err
    from paper_2601_04904_amd import solver as S
    from paper_2601_04904_amd.synth import gen_problem
    probs = [gen_problem(2, b, 0, 0.3, 0.05, b) for b in sizes]
    dA = [S.DeviceBlocks.from_host(A) for A, _ in probs]
    dB = [S.DeviceBlocks.from_host(B) for _, B in probs]
    XR = [S.DeviceBlocks.empty(A.n, A.b, A.a) for A, _ in probs]
    XL = [S.DeviceBlocks.empty(A.n, A.b, A.a) for A, _ in probs]
    bs = S.BatchSolver([dict(n=A.n, b=A.b, a=A.a) for A, _ in probs])
    bs.solve(dA, dB, XR, XL)
    bs.sync()
    for i, (A, B) in enumerate(probs):
        R, L = oracle.solve_dense(A, B)
        assert rel_err(XR[i].to_host(), R) < 1e-11, i
        assert rel_err(XL[i].to_host(), L) < 1e-11, i
    bs.destroy()


@pytest.mark.parametrize("d", [3, 4, 5, 31, 48, 49, 63, 64, 65, 79, 111, 112, 113, 127, 128, 129, 145, 255, 256, 257,
                               511, 512, 513, 1023])
def test_inverse_shape_edges(torch, d):
    from paper_2601_04904_amd.solver import diag_inverse
    rng = np.random.default_rng(d)
    count = 3 if d <= 300 else 1
    M = crand(rng, count, d, d) / np.sqrt(d)
    M[:, np.arange(d), np.arange(d)] = 0.0                     # no pivot on the diagonal
    M[0] *= 10.0 ** rng.uniform(-3, 3, size=(d, 1))            # rows of different size
    dst, bad = diag_inverse(torch.from_numpy(M).cuda())
    assert bad == -1
    got = dst.cpu().numpy()
    for i in range(count):
        ref = np.linalg.inv(M[i])
        err = np.linalg.norm(got[i] - ref) / np.linalg.norm(ref)
        assert err < 50 * EPS * np.sqrt(d) * np.linalg.cond(M[i]), (i, err)


@pytest.mark.parametrize("d", [40, 100, 120, 200, 300])
def test_inverse_reports_singular(torch, d):
    """A zero column: reported for every kernel shape, the other matrices inverted."""
    from paper_2601_04904_amd.solver import diag_inverse
    rng = np.random.default_rng(d)
    M = crand(rng, 3, d, d) + np.eye(d)
    M[1][:, d // 2] = 0.0
    M[1][d // 2, :] = 0.0
    dst, bad = diag_inverse(torch.from_numpy(M).cuda())
    assert bad == 1
    got = dst.cpu().numpy()
    for i in (0, 2):
        ref = np.linalg.inv(M[i])
        assert np.linalg.norm(got[i] - ref) / np.linalg.norm(ref) < 1e-10


@pytest.mark.parametrize("n,b,a,P", [(1, 1, 0, 1), (2, 15, 1, 1), (5, 16, 17, 1), (4, 17, 0, 1), (6, 33, 31, 2),
                                     (5, 48, 0, 1), (4, 64, 64, 1), (16, 5, 3, 8), (24, 20, 9, 6)])
@pytest.mark.parametrize("antih", [False, True])
def test_fused_tile_edges(torch, n, b, a, P, antih):
    """BT_FUSED at tile edges of its products, with more products in a level than
    one step holds (many partitions), alone and beside enough copies of itself
    that the instances share CUs."""
    import oracle
    from tests._util import rel_err
    from paper_2601_04904_amd import solver as S
    from paper_2601_04904_amd.synth import gen_problem
    A, B = gen_problem(n, b, a, 0.3, 0.05, 31 * n + b)
    R, L = oracle.solve_dense(A, B)
    flags = S.BT_FUSED | (S.BT_SIGMA_ANTIHERMITIAN if antih else 0)
    dA, dB = S.DeviceBlocks.from_host(A), S.DeviceBlocks.from_host(B)
    for count in (1, 300):
        out = [(S.DeviceBlocks.empty(n, b, a), S.DeviceBlocks.empty(n, b, a)) for _ in range(count)]
        bs = S.BatchSolver([dict(n=n, b=b, a=a, partitions=P, flags=flags)] * count)
        bs.solve([dA] * count, [dB] * count, [x[0] for x in out], [x[1] for x in out])
        bs.sync()
        for i in (0, count - 1):
            assert rel_err(out[i][0].to_host(), R) < 1e-11
            assert rel_err(out[i][1].to_host(), L) < 1e-11
        bs.destroy()


def test_products_of_different_length_in_a_launch(torch):
    """Instances of very different block sizes and partition counts in one batch:
    launches that mix one-term and six-term products of 3 to 130 rows, so that
    tile orders have several classes and padding."""
    import oracle
    from tests._util import rel_err
    from paper_2601_04904_amd import solver as S
    from paper_2601_04904_amd.synth import gen_problem
    specs = [(7, 130, 9, 3), (5, 65, 64, 1), (9, 3, 2, 4), (4, 33, 0, 2), (6, 64, 31, 2)]
    probs = [gen_problem(n, b, a, 0.3, 0.05, 11 + b) for n, b, a, _ in specs]
    dA = [S.DeviceBlocks.from_host(A) for A, _ in probs]
    dB = [S.DeviceBlocks.from_host(B) for _, B in probs]
    XR = [S.DeviceBlocks.empty(n, b, a) for n, b, a, _ in specs]
    XL = [S.DeviceBlocks.empty(n, b, a) for n, b, a, _ in specs]
    bs = S.BatchSolver([dict(n=n, b=b, a=a, partitions=P) for n, b, a, P in specs])
    bs.solve(dA, dB, XR, XL)
    bs.sync()
    for i, (A, B) in enumerate(probs):
        R, L = oracle.solve_dense(A, B)
        assert rel_err(XR[i].to_host(), R) < 1e-11, i
        assert rel_err(XL[i].to_host(), L) < 1e-11, i
    bs.destroy()
