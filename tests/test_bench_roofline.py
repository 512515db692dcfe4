"""bench.py's roofline of the sweep kernel comes from runs of that kernel (no GPU needed).

A run in the resident form has no sweep-kernel launches: where the default run
takes it, the launch chain is timed beside it, with its groups chosen.
"""
import json
import sys

import pytest

torch = pytest.importorskip("torch")

from test_bench_guard import load_bench  # noqa: E402

SITES = 3 * 160 * 480 * 600


def run(resident, ms, groups=3, grid=640):
    return dict(ms_per_sweep=ms, sweeps_per_launch=50, launches=1, warmup_sweeps=50, resident=resident,
                groups=None if resident else groups, grid=None if resident else grid, sites=SITES, ctx_means=None)


@pytest.mark.parametrize("form,fmt", [("batched", "bitpack"), ("batched", "int8"), ("persistent", "bitpack"),
                                      ("plain", "int8")])
def test_figures_of_the_sweep_kernel_are_its_own(monkeypatch, capsys, form, fmt):
    bench = load_bench()
    asked = []

    def run_form(islf, torch_, form, fmt, *a, groups=0, barriers=None, **k):
        asked.append((form, fmt, groups))
        if groups == 1:
            return run(False, 0.080, 1, 2048)
        if groups or (form, fmt) == ("batched", "bitpack"):
            return run(False, 0.090 if fmt == "int8" else 0.060)
        return run(True, 0.0625)     # the resident form

    monkeypatch.setattr(bench, "run_form", run_form)
    monkeypatch.setattr(bench, "committed_valu", lambda fmt: {"issue_us_per_launch": 27.0 if fmt == "bitpack" else 37.0})
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(sys, "argv", ["bench.py", "--form", form, "--fmt", fmt, "--no-aux", "--no-cpu", "--no-configs"])
    bench.main()
    line = json.loads(capsys.readouterr().out)
    r = line["roofline"]
    other = "int8" if fmt == "bitpack" else "bitpack"
    assert r["launch_ms"] == 0.04 and r["workgroups"] == 2048
    for q, f in ((r, fmt), (r["other_format_" + other], other)):
        if "grouped_wave" in q:
            wave = 0.045 if f == "int8" else 0.03
            assert q["grouped_wave"]["wave_ms"] == wave
            assert q["grouped_wave"]["valu_issue_frac"] == round((27.0 if f == "bitpack" else 37.0) / (wave * 1e3), 3) < 1
    assert ("grouped_wave" in r) == (form == "batched")
    assert r["grouped_wave_is_headline_form"] == ((form, fmt) == ("batched", "bitpack"))
    resident = (form, fmt) != ("batched", "bitpack")
    assert line["config"]["resident"] == resident and (line["config"]["groups"] is None) == resident
    assert line["value"] == round(SITES / ((0.0625 if resident else 0.06) * 1e6), 2)
    assert r["other_format_" + other]["batched_form_is_resident"] == (other == "int8")


def test_a_resident_run_is_no_sweep_kernel():
    bench = load_bench()
    with pytest.raises(AssertionError):
        bench.roofline_of("int8", run(True, 0.06), None)
    with pytest.raises(AssertionError):
        bench.roofline_of("int8", run(False, 0.08, 1), run(True, 0.06))
