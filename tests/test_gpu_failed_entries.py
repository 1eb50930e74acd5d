"""Entries that the guard of a default product leaves to the plain kernels, in
tiles of every size, split along k and not, in square, triangular, long and complex
products, with all, some or few entries of a tile failing.

Where whole tiles fail and the plain product runs unsplit in the same tiles, the
result is its bit for bit; otherwise it is within the sum of the two bounds,
k + 8 units of 2^-104 (|alpha| |A||B| + |beta| |C|) each.  Every product runs
several times on one handle, on two streams, with the same bits."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, entries_mask, host, op_abs
from oracle.compare import bits, componentwise

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    import torch
    from paper_2109_13406_amd import binding as b
    handle = b.mpdd_create()
    yield handle
    torch.cuda.synchronize()
    b.mpdd_destroy(handle)


def _edit(what, A, B):
    """Edit (hi, lo) views of op(A) (m x k) and op(B) (k x n) in place."""
    m, k = A[0].shape
    if what == "graded":                    # every entry's bound fails
        s = 2.0 ** np.round(np.linspace(0, -100, k))
        for v in A:
            v *= s
        for v in B:
            v /= s[:, None]
    else:                                   # rows of one dominant entry
        rows = {"all rows": range(m), "every third row": range(0, m, 3),
                "two rows": (3, m - 2), "upper half": range(m // 2)}[what]
        for i in rows:
            A[0][i, (7 * i) % k], A[1][i, (7 * i) % k] = 2.0 ** 30, 0.0


def _call(h, case, ops, opts, stream=None):
    from paper_2109_13406_amd import binding as b
    C = [x.clone() for x in ops["C"]]
    if "uplo" in case:
        args = (case["uplo"], case["trans"], case["n"], case["k"], case["alpha"], ops["A"],
                case["lda"], case["beta"], C, case["ldc"])
        rc = (b.mpdd_Rsyrk_ex(h, opts, *args, stream=stream) if opts else
              b.mpdd_Rsyrk(h, *args, stream=stream))
    else:
        args = (case["transa"], case["transb"], case["m"], case["n"], case["k"], case["alpha"],
                ops["A"], case["lda"], ops["B"], case["ldb"], case["beta"], C, case["ldc"])
        rc = (b.mpdd_Rgemm_ex(h, opts, *args, stream=stream) if opts else
              b.mpdd_Rgemm(h, *args, stream=stream))
    assert rc == 0
    return C


def _check(h, case, m, n, tri, exact):
    import torch
    from paper_2109_13406_amd import binding as b
    k = case["k"]
    ops = {x: dev(case[x]) for x in "ABC" if x in case}
    P = host(_call(h, case, ops, dict(algo=b.MPDD_PLAIN)))
    streams = [None, torch.cuda.Stream(), None]
    torch.cuda.synchronize()
    G = []
    for s in streams:
        G.append(_call(h, case, ops, None, s))
        torch.cuda.synchronize()
    G = [host(x) for x in G]
    for g in G[1:]:
        assert all(np.array_equal(bits(x), bits(y)) for x, y in zip(g, G[0]))
    idx = entries_mask(m, n, case["ldc"], tri)
    if exact:
        for p in range(2):
            assert np.array_equal(bits(G[0][p])[idx], bits(P[p])[idx])
    else:
        i, j = np.meshgrid(np.arange(m), np.arange(n), indexing="ij")
        sel = np.ones_like(i, bool) if tri is None else (i <= j if tri == "U" else i >= j)
        absab = (op_abs(case, "A") @ op_abs(case, "B"))[sel]
        c = componentwise(G[0][0][idx], G[0][1][idx], P[0][idx], P[1][idx], absab, case["alpha"],
                          case["beta"], case["C"][0][idx])
        assert c <= 2 * (k + 8)
    rest = np.ones(G[0][0].shape[0], bool)
    rest[idx] = False
    for p in range(2):
        assert np.array_equal(bits(G[0][p])[rest], bits(case["C"][p])[rest])


# (route, plain tile and split): all the built-in choice has
GEMM = [(600, 600, 600, (1, 2, 2)), (640, 640, 640, (1, 2, 1)), (384, 384, 1024, (1, 5, 4)),
        (1024, 1024, 1024, (1, 4, 4)), (2048, 2048, 400, (1, 4, 1)),
        (1025, 383, 1000, (1, 2, 4)), (33, 2000, 3000, (2, 5, 2)),
        (1031, 64, 4001, (2, 2, 32)), (16, 4096, 4096, (2, 4, 16))]


@pytest.mark.parametrize("what", ["graded", "all rows", "every third row", "two rows",
                                  "upper half"])
@pytest.mark.parametrize("m,n,k,plan", GEMM)
def test_failed_entries_gemm(h, m, n, k, plan, what):
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_OP_GEMM, m, n, k) == plan
    ta, tb = ("NN", "NT", "TN", "TT")[(m + len(what)) % 4]
    case = W.gemm_case(7900 + m, ta, tb, m, n, k)
    A = [W.view(x, *((m, k) if ta == "N" else (k, m)), case["lda"]) for x in case["A"]]
    B = [W.view(x, *((k, n) if tb == "N" else (n, k)), case["ldb"]) for x in case["B"]]
    _edit(what, [v if ta == "N" else v.T for v in A], [v if tb == "N" else v.T for v in B])
    # whole 64 x 64 blocks, and a plain product that is not split either: its tile
    whole = m % 64 == 0 and n % 64 == 0 and plan[2] == 1
    _check(h, case, m, n, None, exact=whole and what in ("graded", "all rows"))


SYRK = [(1100, 513, (1, 5, 1)), (1280, 640, (1, 5, 1)), (2048, 512, (1, 2, 1)),
        (640, 2100, (1, 2, 2))]


@pytest.mark.parametrize("what", ["all rows", "every third row", "two rows"])
@pytest.mark.parametrize("uplo,trans", ["UN", "LT"])
@pytest.mark.parametrize("n,k,plan", SYRK)
def test_failed_entries_syrk(h, n, k, plan, uplo, trans, what):
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_OP_SYRK, n, n, k) == plan
    case = W.syrk_case(7950 + n, uplo, trans, n, k)
    A = [W.view(x, *((n, k) if trans == "N" else (k, n)), case["lda"]) for x in case["A"]]
    _edit(what, [v if trans == "N" else v.T for v in A], None)
    _check(h, case, n, n, uplo, exact=False)


@pytest.mark.parametrize("what", ["graded", "all rows", "every third row"])
@pytest.mark.parametrize("m,n,k", [(512, 512, 512), (260, 130, 3000)])
def test_failed_entries_cgemm(h, m, n, k, what):
    import torch
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_TEST_CGEMM, m, n, k)[0] == 1
    c = W.cgemm_case(7970 + m, "N", "C", m, n, k)
    A = [W.view(x, m, k, c["lda"]) for x in c["A"]]
    B = [W.view(x, n, k, c["ldb"]).T for x in c["B"]]
    _edit(what, A[:2], B[:2])
    _edit(what, A[2:], B[2:])
    absa, absb = np.hypot(A[0], A[2]), np.hypot(B[0], B[2])
    dA, dB, dC = ([torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c[y]] for y in "ABC")
    out = []
    for opts in (dict(algo=b.MPDD_PLAIN), None, None):
        C = [x.clone() for x in dC]
        args = ("N", "C", m, n, k, c["alpha"], dA, c["lda"], dB, c["ldb"], c["beta"], C, c["ldc"])
        assert (b.mpdd_Cgemm_ex(h, opts, *args) if opts else b.mpdd_Cgemm(h, *args)) == 0
        torch.cuda.synchronize()
        out.append([W.view(x.cpu().numpy(), m, n, c["ldc"]) for x in C])
    P, G, G2 = out
    size = lambda s: np.hypot(s[0][0], s[1][0])
    C0 = [W.view(x, m, n, c["ldc"]) for x in c["C"]]
    unit = 2.0 ** -104 * (size(c["alpha"]) * (absa @ absb) +
                          size(c["beta"]) * np.hypot(C0[0], C0[2]))
    for q in (0, 2):
        d = np.abs((G[q] - P[q]) + (G[q + 1] - P[q + 1]))
        assert np.max(d / unit) <= 4 * (k + 8)          # two products a part
        assert np.array_equal(bits(G[q]), bits(G2[q]))
        assert np.array_equal(bits(G[q + 1]), bits(G2[q + 1]))


def _exact_errors(A, B, got, rows, cols):
    """Errors of got's sampled entries against the exact products, in units of
    2^-104 (|A||B|)_ij: pairs as integers times 2^-S."""
    S = 300
    ints = lambda hi, lo: [int(h * 2.0 ** 200) * (1 << (S - 200)) + int(l * 2.0 ** 200) *
                           (1 << (S - 200)) for h, l in zip(hi, lo)]
    out = []
    for i, j in zip(rows, cols):
        a, b = ints(A[0][i], A[1][i]), ints(B[0][:, j], B[1][:, j])
        exact = sum(x * y for x, y in zip(a, b))
        size = sum(abs(x * y) for x, y in zip(a, b))
        g = ints([got[0][i, j]], [got[1][i, j]])[0] << S
        out.append((g - exact) * (1 << 104) / size)
    return np.array(out)


@pytest.mark.parametrize("m,n,k", [(1024, 1024, 1024), (600, 600, 600), (700, 200, 2000),
                                   (1031, 64, 4001)])
def test_refused_entries_round_no_more_than_the_plain_product(h, m, n, k):
    """Rows of one dominant entry above many small ones: root mean square over 400
    sampled entries, with 15 % for the sampling (three times the spread of the
    ratio of two such means)."""
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_OP_GEMM, m, n, k)[0] > 0
    case = W.gemm_case(7990, "N", "N", m, n, k, beta_zero=True)
    case["alpha"] = (1.0, 0.0)
    A = [W.view(x, m, k, case["lda"]) for x in case["A"]]
    B = [W.view(x, k, n, case["ldb"]) for x in case["B"]]
    # (sum |x| / 2^sigma < 4 and sum (x / 2^sigma)^2 < 2 for every row)
    for v in A:
        v *= 2.0 ** -np.ceil(np.log2(k / 2.0))
    i = np.arange(m)
    A[0][i, (7 * i) % k], A[1][i, (7 * i) % k] = 0.77, 0.77 * 2.0 ** -54
    rng = np.random.default_rng(5)
    rows, cols = rng.integers(0, m, 400), rng.integers(0, n, 400)
    rms = []
    for opts in (dict(algo=b.MPDD_PLAIN), None):
        C = host(_call(h, case, {x: dev(case[x]) for x in "ABC"}, opts))
        C = [W.view(x, m, n, case["ldc"]) for x in C]
        rms.append(np.sqrt(np.mean(_exact_errors(A, B, C, rows, cols) ** 2)))
    assert rms[1] <= 1.15 * rms[0], rms


@pytest.mark.parametrize("m,n,k", [(200, 200, 200), (200, 96, 130), (72, 131, 300)])
def test_failed_entries_qgemm(h, m, n, k):
    """All entries failed (spread operands): tiles with more than 96 of them, the
    narrow ones at the edges included, are the plain kernel's bit for bit."""
    import torch
    from paper_2109_13406_amd import binding as b
    assert b.mpdd_test_route(b.MPDD_TEST_QGEMM, m, n, k)[0] == 1
    c = W.qgemm_case(7995, "N", "N", m, n, k)
    s = 2.0 ** np.round(np.linspace(0, -100, k))
    for x in c["A"]:
        W.view(x, m, k, c["lda"])[:] *= s
    for x in c["B"]:
        W.view(x, k, n, c["ldb"])[:] /= s[:, None]
    dA, dB, dC = ([torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in c[y]] for y in "ABC")
    out = []
    for opts in (dict(algo=b.MPDD_PLAIN), None):
        C = [x.clone() for x in dC]
        assert b.mpdd_Qgemm(h, "N", "N", m, n, k, c["alpha"], dA, c["lda"], dB, c["ldb"],
                            c["beta"], C, c["ldc"], opts=opts) == 0
        torch.cuda.synchronize()
        out.append([W.view(x.cpu().numpy(), m, n, c["ldc"]) for x in C])
    tile = lambda size: np.minimum(32, size - np.arange(size) // 32 * 32)
    whole = tile(m)[:, None] * tile(n)[None, :] > 96
    for p, g in zip(*out):
        assert np.array_equal(bits(p[whole]), bits(g[whole]))
    d = sum(g - p for p, g in zip(*out))
    unit = 2.0 ** -209 * (abs(c["alpha"][0]) *
                          (np.abs(W.view(c["A"][0], m, k, c["lda"])) @
                           np.abs(W.view(c["B"][0], k, n, c["ldb"]))) +
                          abs(c["beta"][0]) * np.abs(W.view(c["C"][0], m, n, c["ldc"])))
    assert np.max(np.abs(d) / unit) <= 2 * (k + 8)
