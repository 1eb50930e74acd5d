"""A group whose launch fails after some of its kernels were enqueued: every
request of it returns the error, and none runs a second time (with beta != 0 a
second run would update C twice)."""
import numpy as np
import pytest

from paper_2109_13406_amd import binding as b
from test_server_cpu import _gemm, server_factory  # noqa: F401


@pytest.mark.parametrize("size", [2, 6])
def test_partly_launched_group_is_not_run_again(server_factory, size):  # noqa: F811
    # four long requests hold the slots; the others then go as one group
    s = server_factory(rate=1e12, latency=0.2)
    held = [b.mpdd_server_submit(s, _gemm(40, 40, 40)) for _ in range(4)]
    group = [b.mpdd_server_submit(s, _gemm(30, 30, 30, inject=3 if i == 1 else 0))
             for i in range(size)]
    assert all(b.mpdd_server_wait(s, t)[0] == 0 for t in held)
    got = [b.mpdd_server_wait(s, t) for t in group]
    assert [info for info, _ in got] == [b.MPDD_ERR_HIP] * size
    assert len({tm["group"] for _, tm in got}) == 1
    st = b.mpdd_server_get_stats(s)
    assert st["groups"] == 5 and st["failed"] == size
    assert st["inflight_bytes"] == 0 and st["inflight_requests"] == 0
    # the server keeps serving
    assert b.mpdd_server_wait(s, b.mpdd_server_submit(s, _gemm(30, 30, 30)))[0] == 0


def test_failure_before_any_launch_is_still_isolated(server_factory):  # noqa: F811
    s = server_factory(rate=1e12, latency=0.05)
    held = [b.mpdd_server_submit(s, _gemm(40, 40, 40)) for _ in range(4)]
    group = [b.mpdd_server_submit(s, _gemm(30, 30, 30, inject=1 if i == 2 else 0))
             for i in range(5)]
    infos = [b.mpdd_server_wait(s, t)[0] for t in held + group]
    assert infos == [0] * 6 + [b.MPDD_ERR_HIP] + [0] * 2


@pytest.mark.gpu
@pytest.mark.parametrize("alone", [False, True])
def test_partly_launched_group_updates_c_once(alone):
    import torch
    import workloads as W
    from gpu_util import dev, gemm_gpu, host
    from oracle.compare import bits
    # one request per served tile shape, and large ones that hold the slots
    shapes = [(64, 64, 64)] if alone else [(64, 64, 64), (200, 300, 90), (700, 650, 600)]
    cases = [W.gemm_case(7700 + i, "N", "T", *x) for i, x in enumerate(shapes)]
    assert all(c["beta"] != (0.0, 0.0) for c in cases)
    big = W.gemm_case_device(7790, "N", "N", 2048, 2048, 1024, padded=False)
    h = b.mpdd_create()
    s = b.mpdd_server_create(h, 1 << 36, 64)
    try:
        ops = [{x: dev(c[x]) for x in "ABC"} for c in cases]
        torch.cuda.synchronize()

        def request(c, o, inject=0):
            return b.make_request(b.MPDD_OP_GEMM, c["transa"], c["transb"], c["m"], c["n"],
                                  c["k"], c["alpha"], o["A"], c["lda"], o["B"], c["ldb"],
                                  c["beta"], o["C"], c["ldc"], inject=inject)
        held = []
        if not alone:
            for _ in range(4):
                C = [torch.zeros_like(x) for x in big["C"]]
                held.append((b.mpdd_server_submit(s, request(big, dict(big, C=C))), C))
        group = [b.mpdd_server_submit(s, request(c, o, inject=3 if i == 0 else 0))
                 for i, (c, o) in enumerate(zip(cases, ops))]
        got = [b.mpdd_server_wait(s, t) for t in group]
        assert all(b.mpdd_server_wait(s, t)[0] == 0 for t, _ in held)
        torch.cuda.synchronize()
        for c, o, (info, tm) in zip(cases, ops, got):
            G = host(o["C"])
            _, once = gemm_gpu(h, c, opts=dict(tile_id=tm["tile"], splitk=1))
            same = [np.array_equal(bits(g), bits(x)) for g, x in zip(G, once)]
            if info == 0:                  # went in another group
                assert tm["group"] != got[0][1]["group"]
            else:
                assert info == b.MPDD_ERR_HIP and tm["group"] == got[0][1]["group"]
            assert all(same)
        assert got[0][0] == b.MPDD_ERR_HIP
    finally:
        b.mpdd_server_destroy(s)
        b.mpdd_destroy(h)
