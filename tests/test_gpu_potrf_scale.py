"""Rpotrf on matrices near the ends of the exponent range: Cholesky commutes with
a scaling of rows and columns by powers of two, and every operation of it does as
long as nothing under- or overflows, so the factor of D A D is D L bit for bit
(pivots up to 2^1008 and down to 2^-752, diagonals spread over 2^1780)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, host
from oracle.compare import bits

pytestmark = pytest.mark.gpu

SCALES = {"large": lambda n: np.full(n, 500), "small": lambda n: np.full(n, -380),
          "falling": lambda n: np.round(np.linspace(490, -400, n)).astype(int),
          "rising": lambda n: np.round(np.linspace(-400, 490, n)).astype(int),
          "mixed": lambda n: np.where(np.arange(n) % 3 == 0, 491, -399)}


def _factor(n, uplo, scale, fail_at):
    from paper_2109_13406_amd import binding as b
    c = W.spd_case(7500 + n, n, uplo, fail_at=fail_at)
    e = scale[:, None] + scale[None, :]
    A = [x.copy() for x in c["A"]]
    for x in A:
        v = W.view(x, n, n, c["lda"])
        v[:] = np.ldexp(v, e)
    D = dev(A)
    h = b.mpdd_create()
    try:
        rc, info = b.mpdd_Rpotrf(h, uplo, n, D, c["lda"])
        G = host(D)
    finally:
        b.mpdd_destroy(h)
    assert rc == 0 and info == (fail_at or 0)
    G = [W.view(x, n, n, c["lda"]) for x in G]
    return [x.T for x in G] if uplo == "U" else G     # lower view


@pytest.mark.parametrize("scale", list(SCALES))
@pytest.mark.parametrize("uplo", "LU")
@pytest.mark.parametrize("n,fail_at", [(61, None), (150, None), (300, None), (150, 100)])
def test_factor_scales_with_its_rows(uplo, n, fail_at, scale):
    s = SCALES[scale](n)
    L0 = _factor(n, uplo, np.zeros(n, int), fail_at)
    L1 = _factor(n, uplo, s, fail_at)
    last = fail_at or n                       # columns to compare
    i, j = np.tril_indices(n)
    keep = (j < last - 1) if fail_at else (j < n)
    if fail_at:
        # the finished columns of the blocks up to the failing one, and the pivot
        keep &= i < (fail_at - 1) // 64 * 64 + 64
        p = fail_at - 1
        assert L0[0][p, p] < 0.0
        assert np.ldexp(L1[0][p, p], -2 * int(s[p])) == L0[0][p, p]
    i, j = i[keep], j[keep]
    for a, g in zip(L0, L1):
        assert np.array_equal(bits(np.ldexp(g[i, j], -s[i])), bits(a[i, j]))
