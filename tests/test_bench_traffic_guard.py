"""bench.py reports recorded HBM traffic only for the sources it was counted on:
every source that holds the kernels or the rules of a dense H_eff product
changes the hash it compares."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load(tmp_path):
    spec = importlib.util.spec_from_file_location("bench_guard", os.path.join(ROOT, "bench.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    src = tmp_path / "paper_1501_05504_amd" / "csrc"
    src.mkdir(parents=True)
    here = os.path.join(ROOT, "paper_1501_05504_amd", "csrc")
    for name in os.listdir(here):
        (src / name).write_bytes(open(os.path.join(here, name), "rb").read())
    b.ROOT = str(tmp_path)
    return b, src


@pytest.mark.parametrize("name", ["gemm.hip", "direct.hip", "mfma_tile.h", "kernels.hip", "ops.hip"])
def test_a_changed_source_changes_the_hash(tmp_path, name):
    b, src = load(tmp_path)
    before = b.gemm_source_sha()
    with open(src / name, "a") as f:
        f.write("\n")
    assert b.gemm_source_sha() != before
