"""Default products whose way is asserted: the guarded modular form at its smallest
k, at the edges of its tiles and of the steps of the route's allowance, both
triangles, C only written; and the plain kernels at large sizes, where only
MPDD_PLAIN reaches them.

Errors are against exact integer products of sampled entries, in units of 2^-104
(|A||B|)_ij.  An entry that passes the guard is within k^(1/2) units of grid rounding
plus 2 of the reconstruction's; uniform data pass everywhere, and there the form
is closer to the exact product than the plain kernels are.  A plain entry is within
k + 4."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, entries_mask, gemm_gpu, host, syrk_gpu
from oracle.compare import bits
from test_gpu_failed_entries import _exact_errors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    import torch
    from paper_2109_13406_amd import binding as b
    handle = b.mpdd_create()
    yield handle
    torch.cuda.synchronize()
    b.mpdd_destroy(handle)


def _ops(case):
    """(hi, lo) views of op(A) and op(B)."""
    if "uplo" in case:
        n, k = case["n"], case["k"]
        s = (n, k) if case["trans"] == "N" else (k, n)
        A = [W.view(x, *s, case["lda"]) for x in case["A"]]
        A = A if case["trans"] == "N" else [v.T for v in A]
        return A, [v.T for v in A]
    m, n, k = case["m"], case["n"], case["k"]
    A = [W.view(x, *((m, k) if case["transa"] == "N" else (k, m)), case["lda"])
         for x in case["A"]]
    B = [W.view(x, *((k, n) if case["transb"] == "N" else (n, k)), case["ldb"])
         for x in case["B"]]
    return (A if case["transa"] == "N" else [v.T for v in A],
            B if case["transb"] == "N" else [v.T for v in B])


def _samples(m, n, tri, count, seed):
    rng = np.random.default_rng(seed)
    i, j = rng.integers(0, m, count), rng.integers(0, n, count)
    # the corners too
    i, j = np.append(i, [0, m - 1, m - 1]), np.append(j, [0, 0 if tri != "U" else n - 1, n - 1])
    if tri == "U":
        i, j = np.minimum(i, j), np.maximum(i, j)
    elif tri == "L":
        i, j = np.maximum(i, j), np.minimum(i, j)
    return i, j


def _errors(case, G, m, n, tri=None, count=120):
    A, B = _ops(case)
    i, j = _samples(m, n, tri, count, 11)
    return _exact_errors(A, B, [W.view(x, m, n, case["ldc"]) for x in G], i, j)


def _rest_untouched(case, G, m, n, tri=None):
    rest = np.ones(G[0].shape[0], bool)
    rest[entries_mask(m, n, case["ldc"], tri)] = False
    for p in range(2):
        assert np.array_equal(bits(G[p])[rest], bits(case["C"][p])[rest])


GEMM = [("NN", 2048, 1500, 350), ("TN", 2049, 1600, 399), ("NT", 1025, 769, 400),
        ("TT", 640, 577, 513), ("NT", 641, 640, 1025), ("TN", 2049, 511, 640)]


@pytest.mark.parametrize("op,m,n,k", GEMM)
@pytest.mark.parametrize("dist", ["uniform", "wide"])
def test_guarded_gemm_takes_its_route(h, op, m, n, k, dist):
    """C only written, and full of NaN."""
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_OP_GEMM, m, n, k)[0] == 1
    case = W.gemm_case(8700 + m, op[0], op[1], m, n, k, dist=dist, beta_zero=True, c_nan=True)
    case["alpha"] = (1.0, 0.0)
    info, G = gemm_gpu(h, case)
    assert info == 0
    _, P = gemm_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
    idx = entries_mask(m, n, case["ldc"])
    assert not np.isnan(G[0][idx]).any() and not np.isnan(G[1][idx]).any()
    _rest_untouched(case, G, m, n)
    e, p = _errors(case, G, m, n), _errors(case, P, m, n)
    assert np.abs(p).max() <= k + 4
    if dist == "uniform":
        # (none failed: another product than the plain one everywhere but where
        # both happen to round alike)
        assert np.mean(bits(G[1])[idx] == bits(P[1])[idx]) < 0.2
        assert np.abs(e).max() <= np.sqrt(k) + 2
        assert np.sqrt(np.mean(e ** 2)) <= np.sqrt(np.mean(p ** 2))
    else:
        assert np.abs(e).max() <= k + 4          # some are left to the plain kernels


@pytest.mark.parametrize("uplo,trans", ["UN", "UT", "LN", "LT"])
@pytest.mark.parametrize("n,k", [(1800, 400), (1409, 512), (1100, 1024)])
def test_guarded_syrk_takes_its_route(h, uplo, trans, n, k):
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_OP_SYRK, n, n, k)[0] == 1
    case = W.syrk_case(8800 + n, uplo, trans, n, k, beta_zero=True)
    case["alpha"] = (1.0, 0.0)
    info, G = syrk_gpu(h, case)
    assert info == 0
    _, P = syrk_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
    idx = entries_mask(n, n, case["ldc"], uplo)
    assert np.mean(bits(G[1])[idx] == bits(P[1])[idx]) < 0.2
    _rest_untouched(case, G, n, n, uplo)
    e, p = _errors(case, G, n, n, uplo), _errors(case, P, n, n, uplo)
    assert np.abs(e).max() <= np.sqrt(k) + 2
    assert np.sqrt(np.mean(e ** 2)) <= np.sqrt(np.mean(p ** 2))


@pytest.mark.parametrize("op", ["NN", "NT", "TN", "TT"])
@pytest.mark.parametrize("m,n,k", [(2048, 2048, 512), (1100, 1100, 1100), (4100, 70, 3001),
                                   (1025, 2049, 300)])
def test_plain_gemm_large(h, op, m, n, k):
    from paper_2109_13406_amd import binding as b
    case = W.gemm_case(8900 + m, op[0], op[1], m, n, k, beta_zero=True)
    case["alpha"] = (1.0, 0.0)
    info, P = gemm_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
    assert info == 0
    assert np.abs(_errors(case, P, m, n, count=60)).max() <= k + 4
    _rest_untouched(case, P, m, n)


@pytest.mark.parametrize("uplo,trans", ["UN", "UT", "LN", "LT"])
@pytest.mark.parametrize("n,k", [(2048, 512), (1100, 1300)])
def test_plain_syrk_large(h, uplo, trans, n, k):
    from paper_2109_13406_amd import binding as b
    case = W.syrk_case(8950 + n, uplo, trans, n, k, beta_zero=True)
    case["alpha"] = (1.0, 0.0)
    info, P = syrk_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
    assert info == 0
    assert np.abs(_errors(case, P, n, n, uplo, count=60)).max() <= k + 4
    _rest_untouched(case, P, n, n, uplo)


def test_plain_headline_size(h):
    """8192^3 on the plain kernels, the product that the benchmark leads with."""
    import torch
    from paper_2109_13406_amd import binding as b
    n = 8192
    case = W.gemm_case_device(8990, "N", "N", n, n, n)
    zero = (0.0, 0.0)
    C = case["C"]
    assert b.mpdd_Rgemm_ex(h, dict(algo=b.MPDD_PLAIN), "N", "N", n, n, n, (1.0, 0.0), case["A"],
                           case["lda"], case["B"], case["ldb"], zero, C, case["ldc"]) == 0
    torch.cuda.synchronize()
    rng = np.random.default_rng(2)
    i, j = rng.integers(0, n, 24), rng.integers(0, n, 24)
    pick = lambda x, ld, idx, dim: (x[:n * ld].view(n, ld)[:, :n].index_select(
        dim, torch.from_numpy(idx).cuda()).cpu().numpy())
    A = [pick(x, case["lda"], i, 1).T for x in case["A"]]          # rows i
    B = [pick(x, case["ldb"], j, 0).T for x in case["B"]]          # columns j
    G = [np.diag(pick(x, case["ldc"], j, 0).T[i]) for x in C]
    e = [_exact_errors([a[t:t + 1] for a in A], [x[:, t:t + 1] for x in B],
                       [g[t:t + 1, None] for g in G], [0], [0])[0] for t in range(24)]
    assert np.abs(e).max() <= n + 4
