"""The benchmark reports recorded HBM traffic only while everything that a kernel is compiled from is as it was."""

import hashlib
import os
import shutil

import pytest

import bench

CSRC = os.path.join("paper_1707_05882_amd", "csrc")
HEADERS = sorted(f for f in os.listdir(os.path.join(bench.ROOT, CSRC)) if f.endswith(".hpp"))


@pytest.fixture
def tree(tmp_path, monkeypatch):
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


def record(tree, kernel, parts, nbytes):
    h = hashlib.sha256(b"".join((tree / CSRC / p).read_bytes() for p in parts)).hexdigest()[:16]
    with open(tree / "profiles" / "traffic_some.txt", "a") as f:
        f.write(f"{kernel} {h} 1 2 {nbytes}\n")


def test_recorded_traffic_is_reported(tree):
    record(tree, "k_eigen_big", ["k_eigen.hip"] + HEADERS, 5e9)
    record(tree, "k_weak_eigen", ["k_weak.hip"] + HEADERS, 2e9)
    assert bench.measured_traffic(["k_weak_eigen", "k_eigen_lds", "k_eigen_big"], "some") == 7e9
    assert bench.measured_traffic(["k_gemm"], "some") is None


@pytest.mark.parametrize("part", ["k_eigen.hip"] + HEADERS)
def test_any_changed_source_ends_it(tree, part):
    record(tree, "k_eigen_big", ["k_eigen.hip"] + HEADERS, 5e9)
    assert bench.measured_traffic(["k_eigen_big"], "some") == 5e9
    with open(tree / CSRC / part, "a") as f:
        f.write("// changed\n")
    assert bench.measured_traffic(["k_eigen_big"], "some") is None
