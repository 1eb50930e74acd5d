"""A failing pivot in a block column with many rows below its diagonal block:
every workgroup of the panel kernel finds the failure for itself, so the rows
below (and everything else outside the finished columns and the diagonal block)
stay as they were, however late a workgroup starts."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import dev, host
from oracle.compare import EPS_DD, bits

pytestmark = pytest.mark.gpu


# (the first column, inside and the last column of a block; 8 and 16 rows a
# workgroup, the second with more row tiles than workgroups)
@pytest.mark.parametrize("uplo", "LU")
@pytest.mark.parametrize("n,fail_at", [(700, 65), (1500, 100), (2500, 64), (4400, 1)])
def test_rows_below_a_failing_pivot_are_untouched(uplo, n, fail_at):
    from paper_2109_13406_amd import binding as b
    c = W.spd_case(7300 + n, n, uplo, fail_at=fail_at)
    ld = c["lda"]
    A = dev(c["A"])
    h = b.mpdd_create()
    try:
        for rep in range(3):
            for x, a in zip(A, dev(c["A"])):
                x.copy_(a)
            rc, info = b.mpdd_Rpotrf(h, uplo, n, A, ld)
            G = host(A)
            assert rc == 0 and info == fail_at
            G = [W.view(x, n, n, ld) for x in G]
            I = [W.view(x, n, n, ld) for x in c["A"]]
            if uplo == "U":
                G, I = [x.T for x in G], [x.T for x in I]
            j = (fail_at - 1) // 64 * 64           # first column of the failing block
            for g, a in zip(G, I):
                assert np.array_equal(bits(np.ascontiguousarray(g[j + 64:, j:])),
                                      bits(np.ascontiguousarray(a[j + 64:, j:])))
    finally:
        b.mpdd_destroy(h)
    if j == 0:
        return
    # the finished columns hold the factor of the leading minor
    sub = W.spd_case(7300 + n, n, uplo)
    O = [np.asfortranarray(W.view(x, n, n, ld)[:j, :j]).ravel(order="F").copy() for x in sub["A"]]
    assert oracle.rpotrf(uplo, j, O, j) == 0
    O = [W.view(x, j, j, j) for x in O]
    if uplo == "U":
        O = [x.T for x in O]
    t = np.tril_indices(j)
    d = (G[0][:j, :j] - O[0])[t] + (G[1][:j, :j] - O[1])[t]
    assert np.linalg.norm(d) / np.linalg.norm(O[0][t]) / (n * EPS_DD) <= 8.0
