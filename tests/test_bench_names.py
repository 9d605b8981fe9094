"""bench.py names the decode kernel instance that a launch plan runs, and reports recorded HBM traffic for that one only."""
import os
import re

import pytest

import bench
from paper_2504_09936_amd import workloads as W
from tests import gpu_util as U

PROFILES = os.path.join(bench.ROOT, "profiles")


def test_decode_kernel_name():
    assert bench.decode_kernel_name(128, 4, True, 224, 8) == "decode_mfma_kernel<128,4,true,1,8>"
    assert bench.decode_kernel_name(128, 4, True, 256, 8) == "decode_mfma_kernel<128,4,true,1,8>"
    assert bench.decode_kernel_name(128, 8, False, 288, 8) == "decode_mfma_kernel<128,8,false,2,8>"
    assert bench.decode_kernel_name(64, 1, True, 256, 4) == "decode_mfma_kernel<64,1,true,2,4>"
    assert bench.decode_kernel_name(128, 8, True, 896, 4) == "decode_mfma_kernel<128,8,true,0,4>"


def test_decode_kernel_name_by_where_the_splits_meet():
    def mode(*a):
        return int(bench.decode_kernel_name(*a).split(",")[3])
    assert [mode(128, 4, True, per, 8, 1, 64) for per in (64, 256, 288, 512, 544)] == [4, 4, 5, 5, 0]              # unsplit
    assert [mode(128, 4, True, 224, 8, 4, heads) for heads in (64, 8, 36, 2056)] == [1, 1, 6, 6]                    # heads by eights
    assert [mode(128, 4, True, per, 8, 17, 8) for per in (224, 448, 544)] == [6, 2, 3]                              # more than sixteen splits
    assert [mode(128, 4, True, 384, 8, ns, heads) for ns, heads in ((4, 64), (4, 56), (2, 128), (8, 32))] == [7, 2, 7, 2]
    assert [mode(64, 4, True, 384, 8, ns, heads) for ns, heads in ((4, 64), (4, 40), (2, 96), (8, 32))] == [7, 2, 7, 2]
    assert [mode(128, 4, False, 384, 8, ns, heads) for ns, heads in ((4, 40), (2, 128), (8, 32), (9, 8), (4, 36))] == [7, 2, 7, 2, 2]   # attention alone


@pytest.mark.parametrize("name", ["llama3_8b", "llama3_70b"])
def test_recorded_traffic_is_that_of_the_planned_instance(name):
    w = W.CONFIGS[name]
    _, per, waves = U.kk().decode_plan(U.layout_of(w), w.budget + w.period)
    kernel = bench.decode_kernel_name(w.head_dim, w.group, True, per, waves)
    assert bench.traffic_from_profile(name, kernel) is not None
    text = open(os.path.join(PROFILES, f"decode_hbm_traffic_{name}.md")).read()
    assert re.search(r"kernel=(\S+)", text).group(1) == kernel
    assert bench.traffic_from_profile(name, kernel.replace("true", "false")) is None


def test_recorded_traffic_says_whether_its_kernel_has_changed(tmp_path, monkeypatch):
    src, rec = tmp_path / "paper_2504_09936_amd" / "csrc", tmp_path / "profiles"
    src.mkdir(parents=True)
    rec.mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    _written(src, "int a;  // one\n")
    assert not bench.traffic_is_of_this_source("w")                                                   # no record
    (rec / "decode_hbm_traffic_w.md").write_text(
        f"<!-- bench: kernel=k<1> fetch_kib=10 write_kib=1 fetch_factor=2.00 write_factor=1.00 source={bench.decode_source_digest()} -->")
    assert bench.traffic_from_profile("w", "k<1>") == 21 * 1024 and bench.traffic_is_of_this_source("w")
    _written(src, "int  a;\n/* two\n lines */  // three\n")
    assert bench.traffic_is_of_this_source("w")                                                       # comments and spaces alone
    _written(src, "int b;\n")
    assert bench.traffic_from_profile("w", "k<1>") == 21 * 1024 and not bench.traffic_is_of_this_source("w")


def _written(folder, text):
    (folder / "decode_attn.hip").write_text(text)
