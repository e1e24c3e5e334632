"""The sources that a kernel's measured traffic is tied to in bench.py."""
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.HERE, "paper_2303_08879_amd", "csrc")


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SOURCES))
def test_a_kernel_is_tied_to_everything_it_is_compiled_from(kernel):
    files = bench.kernel_source_files(kernel)
    assert any(re.search(rf"\bvoid {kernel}\(", t.decode()) for t in files.values())
    for name, text in files.items():
        for inc in re.findall(r'#include "([^"]+)"', text.decode()):
            assert inc in files or not os.path.exists(os.path.join(CSRC, inc)), (name, inc)
    # the shared matrix-core pieces of the reverse kernels
    if kernel.startswith("k_vjp"):
        assert {"vjp_common.h", "pt_units.h", "fd_device.h", "fd_internal.h"} <= set(files)


def test_hash_follows_an_included_file(monkeypatch):
    files = bench.kernel_source_files("k_vjp_block")
    before = bench.kernel_source_hash("k_vjp_block")
    changed = dict(files, **{"pt_units.h": files["pt_units.h"] + b"\n"})
    monkeypatch.setattr(bench, "kernel_source_files", lambda kernel: changed)
    assert bench.kernel_source_hash("k_vjp_block") != before
