"""Default products of matrices with one dominant entry in every row, as Gram and
Schur matrices and Cholesky factors have: full rows are not rows of few terms, and
take the modular form like any others, whose error is a tenth of the plain
product's on them.  Rows of few terms stay with the plain kernels, whose products
of them round less or not at all."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, entries_mask, gemm_gpu, host
from oracle.compare import bits
from test_gpu_failed_entries import _call, _exact_errors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    import torch
    from paper_2109_13406_amd import binding as b
    handle = b.mpdd_create()
    yield handle
    torch.cuda.synchronize()
    b.mpdd_destroy(handle)


def _set(view, x, rng):
    """A full pair matrix with leading parts x."""
    view[0][:] = x
    view[1][:] = x * 2.0 ** -54 * rng.uniform(-1, 1, x.shape)


def _gram(n, rng):
    g = rng.uniform(-1, 1, (n, n))
    return g @ g.T


def _share_as_plain(h, case, m, n, tri=None):
    """Share of entries whose low parts are the plain kernels'."""
    from paper_2109_13406_amd import binding as b
    ops = {x: dev(case[x]) for x in "ABC" if x in case}
    out = [host(_call(h, case, ops, o)) for o in (dict(algo=b.MPDD_PLAIN), None)]
    idx = entries_mask(m, n, case["ldc"], tri)
    return np.mean(bits(out[0][1])[idx] == bits(out[1][1])[idx])


@pytest.mark.parametrize("which", ["A", "B", "AB"])
@pytest.mark.parametrize("n", [640, 1024])
def test_gram_products_take_the_modular_form(h, n, which):
    from paper_2109_13406_amd import binding as b
    rng = np.random.default_rng(n)
    case = W.gemm_case(8100 + n, "N", "N", n, n, n, beta_zero=True)
    case["alpha"] = (1.0, 0.0)
    A = [W.view(x, n, n, case["lda"]) for x in case["A"]]
    B = [W.view(x, n, n, case["ldb"]) for x in case["B"]]
    if "A" in which:
        _set(A, _gram(n, rng), rng)
    if "B" in which:
        _set(B, _gram(n, rng), rng)
    rows, cols = rng.integers(0, n, 200), rng.integers(0, n, 200)
    rms = []
    for opts in (dict(algo=b.MPDD_PLAIN), None):
        C = host(_call(h, case, {x: dev(case[x]) for x in "ABC"}, opts))
        C = [W.view(x, n, n, case["ldc"]) for x in C]
        rms.append(np.sqrt(np.mean(_exact_errors(A, B, C, rows, cols) ** 2)))
    # grid of 109 bits or more: 0.29 2^-109 (Q_i + Q_j) 2^(sigma + tau) is at most
    # 0.05 units for these, the plain kernels' k^(1/2) 2^-106 |sums| at least 0.13
    assert rms[1] <= 0.4 * rms[0], rms


@pytest.mark.parametrize("n", [768, 1024])
def test_cholesky_factor_products_take_the_modular_form(h, n):
    rng = np.random.default_rng(n + 1)
    L = np.linalg.cholesky(_gram(n, rng) + np.eye(n))
    for which in "AB":
        case = W.gemm_case(8200 + n, "N", "N", n, n, n)
        v = [W.view(x, n, n, case["ld" + which.lower()]) for x in case[which]]
        _set(v, L, rng)
        # (the first rows and last columns of L are of few terms)
        assert _share_as_plain(h, case, n, n) < 0.5


def test_gram_syrk_and_complex(h):
    import torch
    from paper_2109_13406_amd import binding as b
    rng = np.random.default_rng(3)
    n = 1100
    case = W.syrk_case(8300, "L", "N", n, n)
    _set([W.view(x, n, n, case["lda"]) for x in case["A"]], _gram(n, rng), rng)
    assert b.mpdd_test_route(b.MPDD_OP_SYRK, n, n, n)[0] == 1
    assert _share_as_plain(h, case, n, n, "L") < 0.2
    n = 512
    assert b.mpdd_test_route(b.MPDD_TEST_CGEMM, n, n, n)[0] == 1
    c = W.cgemm_case(8301, "N", "N", n, n, n)
    A = [W.view(x, n, n, c["lda"]) for x in c["A"]]
    _set(A[:2], _gram(n, rng), rng)
    _set(A[2:], _gram(n, rng), rng)
    dA, dB, dC = ([torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c[y]] for y in "ABC")
    out = []
    for opts in (dict(algo=b.MPDD_PLAIN), None):
        C = [x.clone() for x in dC]
        args = ("N", "N", n, n, n, c["alpha"], dA, c["lda"], dB, c["ldb"], c["beta"], C, c["ldc"])
        assert (b.mpdd_Cgemm_ex(h, opts, *args) if opts else b.mpdd_Cgemm(h, *args)) == 0
        torch.cuda.synchronize()
        out.append([W.view(x.cpu().numpy(), n, n, c["ldc"]) for x in C])
    for q in (1, 3):
        assert np.mean(bits(out[0][q]) == bits(out[1][q])) < 0.2


@pytest.mark.parametrize("terms", [1, 2, 3])
def test_rows_of_few_terms_stay_plain(h, terms):
    """A few entries of one size a row, above a background 2^-60 of it."""
    m, n, k = 640, 640, 640
    case = W.gemm_case(8400 + terms, "N", "T", m, n, k)
    A = [W.view(x, m, k, case["lda"]) for x in case["A"]]
    for v in A:
        v *= 2.0 ** -60
    i = np.arange(m)
    for t in range(terms):
        A[0][i, (7 * i + 11 * t) % k], A[1][i, (7 * i + 11 * t) % k] = 0.6, 0.0
    assert _share_as_plain(h, case, m, n) == 1.0
