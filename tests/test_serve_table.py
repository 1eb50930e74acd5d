"""The autotuner's choice of served tiles, the shipped table, and the server on
every tile-table entry that it runs."""
import os

import pytest

from paper_2109_13406_amd import autotune as AT
from paper_2109_13406_amd import binding as b

TABLE = os.path.join(os.path.dirname(b.__file__), "tuning", "serve_gfx950.json")


def _res(**us):
    """{t<tile>: microseconds} as the autotuner's results, unsplit, and a faster split."""
    out = [dict(tile=int(t[1:]), splitk=1, seconds=v * 1e-6) for t, v in us.items()]
    return out + [dict(tile=2, splitk=4, seconds=1e-9), dict(tile=0, splitk=1, seconds=1e-9)]


def test_edges_are_the_librarys():
    for tile, edge in zip(AT.SERVE_TILES, AT.SERVE_EDGES):
        assert b.mpdd_tile_info(tile)[:2] == (edge, edge)


@pytest.mark.parametrize("us,small,large", [(dict(t2=10, t4=30, t5=6), 5, 5),
                                            (dict(t2=10, t4=30, t5=9), 5, 2),
                                            (dict(t2=10, t4=11, t5=10), 5, 4),
                                            (dict(t2=9, t4=30, t5=12), 2, 2),
                                            (dict(t2=10, t4=9), 2, 4)])
def test_served_tile_choice(us, small, large):
    assert AT.serve_best(_res(**us), 64, 120)["tile"] == small
    assert AT.serve_best(_res(**us), 256, 256)["tile"] == large
    assert AT.serve_best([r for r in _res(**us) if r["splitk"] > 1], 64, 64) is None


def test_shipped_table_has_every_bucket_and_small_tile():
    with open(TABLE) as f:
        text = f.read()
    want = {(op, tr, AT.bucket(m), AT.bucket(n), AT.bucket(k))
            for op, _, _, m, n, k in AT.serve_shapes()
            for tr in (("NN", "NT", "TN", "TT") if op == "gemm" else ("NT", "TN"))}
    import json
    entries = json.loads(text)["entries"]
    assert {(e["op"], e["trans"], e["mb"], e["nb"], e["kb"]) for e in entries} == want
    served = {e["serve_tile"] for e in entries}
    assert served <= set(AT.SERVE_TILES) and 5 in served
    # the smallest requests are launch latency: the tile whose waves share the terms
    assert all(e["serve_tile"] == 5 for e in entries if max(e["mb"], e["nb"]) <= 6)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", AT.SERVE_TILES)
def test_server_runs_every_served_tile(tile, tmp_path):
    import numpy as np
    import torch
    import workloads as W
    from gpu_util import dev, gemm_gpu, host
    from oracle.compare import bits
    shapes = [(33, 48, 64), (129, 65, 40), (200, 100, 300), (64, 64, 64)]
    entries = [dict(op="gemm", trans="NN", mb=AT.bucket(m), nb=AT.bucket(n), kb=AT.bucket(k),
                    tile=4, splitk=1, serve_tile=tile, dd_gflops=0.0) for m, n, k in shapes]
    path = str(tmp_path / "tune.json")
    AT.write_cache(path, entries)
    h = b.mpdd_create(path)
    s = b.mpdd_server_create(h, 1 << 34, 64)
    try:
        cases = [W.gemm_case(8600 + i, "N", "N", *x) for i, x in enumerate(shapes)]
        ops = [{x: dev(c[x]) for x in "ABC"} for c in cases]
        torch.cuda.synchronize()
        tickets = [b.mpdd_server_submit(s, b.make_request(
            b.MPDD_OP_GEMM, "N", "N", c["m"], c["n"], c["k"], c["alpha"], o["A"], c["lda"],
            o["B"], c["ldb"], c["beta"], o["C"], c["ldc"])) for c, o in zip(cases, ops)]
        for t, c, o in zip(tickets, cases, ops):
            info, tm = b.mpdd_server_wait(s, t)
            assert info == 0 and tm["tile"] == tile
            G = host(o["C"])
            _, want = gemm_gpu(h, c, opts=dict(tile_id=tile, splitk=1))
            for p in range(2):
                assert np.array_equal(bits(G[p]), bits(want[p]))
    finally:
        b.mpdd_server_destroy(s)
        b.mpdd_destroy(h)
