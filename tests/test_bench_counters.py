"""The counters that bench.py quotes belong to the kernel its workload runs: their hash covers that
kernel's source and every header it includes, so no edit of either leaves stale counters accepted."""
import os
import re
import shutil

import pytest

import bench


@pytest.mark.parametrize("srcs,kernel", [(bench.KERNEL_SRCS, "seg_attn.hip"),
                                         (bench.EXT_KERNEL_SRCS, "mq_attn.hip"),
                                         (bench.EQ_KERNEL_SRCS, "equiv.hip")])
def test_counter_hash_covers_the_kernel_and_its_headers(srcs, kernel, tmp_path, monkeypatch):
    todo, need = [kernel], set()
    while todo:
        name = todo.pop()
        if name in need:
            continue
        need.add(name)
        with open(os.path.join(bench.CSRC, name)) as f:
            todo += [h for h in re.findall(r'^#include "([^"]+)"', f.read(), flags=re.M)
                     if os.path.exists(os.path.join(bench.CSRC, h))]
    assert need == set(srcs)
    for name in srcs:
        shutil.copy(os.path.join(bench.CSRC, name), tmp_path)
    before = bench.kernel_hash(srcs)
    monkeypatch.setattr(bench, "CSRC", str(tmp_path))
    assert bench.kernel_hash(srcs) == before
    md = tmp_path / "c.md"
    md.write_text(f"- kernel_source_sha256_16: {before}\n- workload: w\n")
    for name in srcs:
        assert bench.measured_counters("w", str(md), srcs)
        text = (tmp_path / name).read_text()
        (tmp_path / name).write_text(text + "\n")
        assert bench.measured_counters("w", str(md), srcs) is None
        (tmp_path / name).write_text(text)
