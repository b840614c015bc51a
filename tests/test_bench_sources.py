"""Which sources make the bench's stored counters stale (host)."""
import os
import shutil

import bench


def test_counters_depend_on_every_source_of_the_kernel(tmp_path):
    """The headers that the kernel includes and the file that plans its launch count; comments do
    not."""
    files = bench.source_files(bench.KERNEL_SRC)
    for name in ("prefix_bf16.hpp", "prefix_eval.hpp", "prefix.hpp", "made_bf16.hpp", "elocal_internal.hpp", "kernels.hpp",
                 "api.cpp"):
        assert name in files
    csrc = str(tmp_path / "csrc")
    shutil.copytree(bench.CSRC, csrc)
    before = bench.source_hash(bench.KERNEL_SRC, csrc)
    assert before == bench.source_hash(bench.KERNEL_SRC)
    for name in files:
        path = os.path.join(csrc, name)
        with open(path) as f:
            text = f.read()
        with open(path, "w") as f:
            f.write("// a remark\n/* and\nanother */" + text)
        assert bench.source_hash(bench.KERNEL_SRC, csrc) == before, name
        with open(path, "w") as f:
            f.write(text + "\nstatic int another_value = 1;\n")
        assert bench.source_hash(bench.KERNEL_SRC, csrc) != before, name
        with open(path, "w") as f:
            f.write(text)


def test_counters_of_another_batch_or_source_are_not_used(tmp_path):
    path = str(tmp_path / "counters.json")
    with open(path, "w") as f:
        f.write('{"samples": 8, "source_sha256_16": "%s", "hbm_bytes_per_launch": 5}' % bench.source_hash(bench.KERNEL_SRC))
    assert bench.stored_counters(path, bench.KERNEL_SRC, 8)["hbm_bytes_per_launch"] == 5
    assert bench.stored_counters(path, bench.KERNEL_SRC, 9) == {}
    assert bench.stored_counters(path, bench.CONNECT_SRC, 8) == {}
    assert bench.stored_counters(str(tmp_path / "none.json"), bench.KERNEL_SRC, 8) == {}
