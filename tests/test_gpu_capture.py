"""Calls on a stream under capture: default products run the plain kernels as
graph nodes, replayed with eager work between; Rpotrf, which is synchronous, is
refused and leaves the handle, its kept streams and the capture usable."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, entries_mask, gemm_gpu, host
from oracle.compare import bits

pytestmark = pytest.mark.gpu


@pytest.fixture
def h():
    import torch
    from paper_2109_13406_amd import binding as b
    handle = b.mpdd_create()
    yield handle
    torch.cuda.synchronize()
    b.mpdd_destroy(handle)


def test_default_product_under_capture_is_the_plain_one(h):
    import torch
    from paper_2109_13406_amd import binding as b
    m, n, k = 2048, 2048, 512                  # modular when eager; no k-split
    case = W.gemm_case(7800, "N", "N", m, n, k)
    _, P = gemm_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
    _, G = gemm_gpu(h, case)
    idx = entries_mask(m, n, case["ldc"])
    assert not np.array_equal(bits(G[1])[idx], bits(P[1])[idx])
    A, B, C0 = dev(case["A"]), dev(case["B"]), dev(case["C"])
    C = [x.clone() for x in C0]
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        assert b.mpdd_Rgemm(h, "N", "N", m, n, k, case["alpha"], A, case["lda"], B, case["ldb"],
                            case["beta"], C, case["ldc"]) == 0
    for rep in range(3):
        for x, y in zip(C, C0):
            x.copy_(y)
        assert gemm_gpu(h, case)[0] == 0       # eager work between the replays
        g.replay()
        R = host(C)
        for p in range(2):
            assert np.array_equal(bits(R[p])[idx], bits(P[p])[idx])


def test_potrf_is_refused_under_capture(h):
    import torch
    from paper_2109_13406_amd import binding as b
    n = 300
    c = W.spd_case(7801, n, "L")
    A = dev(c["A"])
    assert b.mpdd_Rpotrf(h, "L", n, A, c["lda"]) == (0, 0)
    want = host(A)
    x = torch.zeros(16, device="cuda")
    D, E = dev(c["A"]), dev(c["A"])
    s, other, g = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
        assert b.mpdd_Rpotrf(h, "L", n, D, c["lda"]) == (b.MPDD_ERR_HIP, 0)
        x.add_(1.0)
        # another stream's call meanwhile: the kept streams are not the graph's
        assert b.mpdd_Rpotrf(h, "L", n, E, c["lda"], stream=other) == (0, 0)
    for p in range(2):
        assert np.array_equal(bits(host(E)[p]), bits(want[p]))
    for rep in range(3):
        g.replay()
        assert b.mpdd_Rpotrf(h, "L", n, E, c["lda"])[0] == 0
    torch.cuda.synchronize()
    assert x.tolist() == [3.0] * 16
    for p in range(2):                         # nothing of the refused call ran
        assert np.array_equal(bits(host(D)[p]), bits(c["A"][p]))
