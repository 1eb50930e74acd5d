"""Sections of the benchmark that report a plain form's figures: what they time and
compare with names the plain kernels (a call without options chooses)."""
import types

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def run(monkeypatch):
    import torch
    from paper_2109_13406_amd import binding as b
    import bench
    calls = []

    def record(name):
        real = getattr(b, name)

        def wrapped(h, opts, *args, **kw):
            calls.append((name, opts))
            return real(h, opts, *args, **kw)
        monkeypatch.setattr(b, name, wrapped)
    for name in ("mpdd_Rgemm_ex", "mpdd_Rsyrk_ex", "mpdd_Cgemm_ex"):
        record(name)
    h = b.mpdd_create()
    args = types.SimpleNamespace(n=1024, steps=1, ozaki_kinds="")
    yield bench, b, h, args, torch.cuda.current_stream(), calls
    torch.cuda.synchronize()
    b.mpdd_destroy(h)


def test_split_form_section_compares_with_the_plain_kernels(run, monkeypatch):
    bench, b, h, args, stream, calls = run

    def refused(*a, **kw):
        raise AssertionError("a call without options in the split-form section")
    monkeypatch.setattr(b, "mpdd_Rgemm", refused)
    bench.bench_ozaki(h, args, stream, 1.0)
    assert calls and all(o == dict(algo=b.MPDD_PLAIN) for _, o in calls)


def test_complex_section_names_its_forms(run):
    bench, b, h, args, stream, calls = run
    out = bench.bench_cgemm(h, args, stream)
    assert {"ms_default", "ms_4m", "ms_3m", "ms_split_i8", "ms_split_crt"} <= set(out)
    algos = [o and o["algo"] for _, o in calls]
    assert b.MPDD_PLAIN in algos and None in algos
    # the four plain products' own result
    assert out["ratio_vs_oracle_4m"] != out["ratio_vs_oracle_default"]


def test_qd_section_compares_with_the_plain_kernel(run, monkeypatch):
    bench, b, h, args, stream, calls = run
    seen = []
    real = b.mpdd_Qgemm
    monkeypatch.setattr(b, "mpdd_Qgemm",
                        lambda *a, opts=None, **kw: (seen.append(opts), real(*a, opts=opts, **kw))[1])
    out = bench.bench_qd(h, args, stream)
    assert None in seen and dict(algo=b.MPDD_PLAIN) in seen
    for form in ("split_i8", "split_crt"):
        rec = out[form]
        assert abs(rec["speedup_vs_plain"] - out["plain"]["ms"] / rec["ms"]) < 0.05


def test_syrk_section_gives_the_split_forms_a_plain_time(run, monkeypatch):
    bench, b, h, args, stream, calls = run
    given = []
    monkeypatch.setattr(bench, "bench_syrk_split",
                        lambda h, args, stream, plain_ms, kind: given.append(plain_ms))
    out = bench.bench_syrk(h, args, stream)
    assert ("mpdd_Rsyrk_ex", dict(algo=b.MPDD_PLAIN)) in calls
    assert given == [out["plain_ms"]] * 2 and out["plain_ms"] > out["ms"]
