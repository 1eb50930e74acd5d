"""A tuning table decides the plain kernels' tile and k-split, and the way a call
without options takes is chosen against what they would run: a table with a slow
entry moves a size to the modular form, one with the built-in choice's moves none."""
import numpy as np
import pytest

import workloads as W
from gpu_util import entries_mask, gemm_gpu
from oracle.compare import bits

pytestmark = pytest.mark.gpu

SHAPES = [(192, 192, 4096), (600, 600, 600), (64, 2048, 2048)]


def _table(path, tile, splitk):
    from paper_2109_13406_amd import autotune as AT
    entries = []
    for m, n, k in SHAPES:
        plan = (tile, splitk) if tile is not None else _route(None, m, n, k)[1:]
        for tr in ("NN", "NT", "TN", "TT"):
            entries.append(dict(op="gemm", trans=tr, mb=AT.bucket(m), nb=AT.bucket(n),
                                kb=AT.bucket(k), tile=plan[0], splitk=plan[1], dd_gflops=0.0))
    AT.write_cache(path, entries)
    return path


def _route(h, m, n, k):
    from paper_2109_13406_amd import binding as b
    return b.mpdd_test_route(b.MPDD_OP_GEMM, m, n, k, h=h)


@pytest.mark.parametrize("tile,splitk,modular", [(None, None, (False, True, False)),
                                                 (4, 1, (True, True, True)),
                                                 (0, 4, (False, True, False))])
def test_route_by_the_handles_table(tmp_path, tile, splitk, modular):
    import torch
    from paper_2109_13406_amd import binding as b
    h = b.mpdd_create(_table(str(tmp_path / "tune.json"), tile, splitk))
    try:
        for (m, n, k), route in zip(SHAPES, modular):
            got = _route(h, m, n, k)
            assert (got[0] > 0) == route, (m, n, k, got)
            assert got[1:] == ((tile, splitk) if tile is not None else _route(None, m, n, k)[1:])
            case = W.gemm_case(8500 + m, "N", "N", m, n, k)
            _, G = gemm_gpu(h, case)
            _, P = gemm_gpu(h, case, opts=dict(algo=b.MPDD_PLAIN))
            idx = entries_mask(m, n, case["ldc"])
            assert np.array_equal(bits(G[1])[idx], bits(P[1])[idx]) == (not route)
    finally:
        torch.cuda.synchronize()
        b.mpdd_destroy(h)
