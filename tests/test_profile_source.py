"""The digest that ties committed counters to a kernel source covers every project header the span kernels
include: counters taken before a change in any of them must not pass as current."""
import os
import re
import shutil

import bench

CSRC = os.path.join("paper_2609_32308_amd", "csrc")


def included(name):
    found, todo = set(), [name]
    while todo:
        f = todo.pop()
        if f not in found:
            found.add(f)
            with open(os.path.join(bench.ROOT, CSRC, f)) as fh:
                todo += re.findall(r'#include "(sd_\w+\.h)"', fh.read())
    return found


def test_digest_follows_every_included_file(tmp_path, monkeypatch):
    files = included("sd_kernels.hip")
    assert {"sd_kernels.hip", "sd_internal.h", "sd_devutil.h"} <= files
    shutil.copytree(os.path.join(bench.ROOT, CSRC), tmp_path / CSRC)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_source_sha()
    for f in sorted(files):
        path = tmp_path / CSRC / f
        text = path.read_text()
        path.write_text(text + "\n")
        assert bench.kernel_source_sha() != before, f
        path.write_text(text)
        assert bench.kernel_source_sha() == before
