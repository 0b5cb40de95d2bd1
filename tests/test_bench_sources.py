"""Which counter summaries the bench accepts (CPU only): those taken on every
source that decides a sweep's traffic, and made from complete collections."""
import json
import os
import shutil

import pytest

import bench
from test_bench_tools import OTHER, SWEEP, _csv

VARS = "void (anonymous namespace)::k_vars<float>(unsigned int const*, float const*)"
COPY = "__amd_rocclr_copyBuffer"


@pytest.fixture
def tree(tmp_path, monkeypatch):
    src = tmp_path / "paper_2310_08230_amd" / "csrc"
    src.mkdir(parents=True)
    (tmp_path / "profiles").mkdir()
    for f in bench.SWEEP_SOURCES:
        shutil.copy(os.path.join(bench.ROOT, "paper_2310_08230_amd", "csrc", f), src)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


def collect(tree, sweep=(SWEEP, VARS), copy=COPY):
    for c, v in (("FETCH_SIZE", 800.0), ("WRITE_SIZE", 1100.0)):
        _csv(tree / c, c, [(name, v) for name in sweep] * 3)
        _csv(tree / (c + "_copy"), c, [(copy, 262144.0)] * 3)
    return [str(tree / f) for f in ("FETCH_SIZE", "WRITE_SIZE", "FETCH_SIZE_copy", "WRITE_SIZE_copy")]


@pytest.mark.parametrize("changed", ["dual.hip", "layout.hip", "dm_internal.h"])
def test_any_changed_source_withdraws_the_figures(tree, changed):
    name = "sweep_plain_fp32_500_hbm_traffic.json"
    out = tree / "profiles" / name
    bench.summarize_counters(*collect(tree), str(out), 1 << 28, two_passes=True)
    assert bench._traffic(name) == (800 + 1100) * 2 * 1024
    shutil.copy(out, tree / "profiles" / "sweep_smoothed_t0.1_1000_valu.json")
    assert bench._smoothed_valu() is not None
    with open(tree / "paper_2310_08230_amd" / "csrc" / changed, "a") as f:
        f.write("\n// changed\n")
    assert bench._traffic(name) is None and bench._smoothed_valu() is None


def test_a_summary_of_one_source_is_not_enough(tree):
    name = "sweep_plain_fp32_500_hbm_traffic.json"
    out = tree / "profiles" / name
    bench.summarize_counters(*collect(tree), str(out), 1 << 28, two_passes=True)
    rec = json.load(open(out))
    del rec["sources_sha256"]   # as before the other two were looked at
    json.dump(rec, open(out, "w"))
    assert bench._traffic(name) is None


@pytest.mark.parametrize("sweep,copy,two", [((VARS,), COPY, False), ((SWEEP,), COPY, True), ((OTHER, VARS), COPY, True),
                                            ((SWEEP, VARS), "other", True)])
def test_incomplete_collections_are_refused(tree, sweep, copy, two):
    out = tree / "profiles" / "t.json"
    with pytest.raises(ValueError):
        bench.summarize_counters(*collect(tree, sweep, copy), str(out), 1 << 28, two_passes=two)
    assert not out.exists()
