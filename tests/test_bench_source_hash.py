"""The hash that ties the committed traffic figure to its kernels covers every file
that the inner operator's element kernel is made of."""
import importlib.util
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["kernels.hip", "vec.hip", "device.hpp", "nlth_impl.hpp"])
def test_hash_changes_with_each_source(tmp_path, name):
    shutil.copy(os.path.join(ROOT, "bench.py"), tmp_path)
    csrc = tmp_path / "paper_2604_02755_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_2604_02755_amd", "csrc"), csrc)
    spec = importlib.util.spec_from_file_location("bench_copy", tmp_path / "bench.py")
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.ROOT = str(tmp_path)
    before = mod.kernel_source_hash()
    with open(csrc / name, "a") as fh:
        fh.write("// \n")
    assert mod.kernel_source_hash() != before
