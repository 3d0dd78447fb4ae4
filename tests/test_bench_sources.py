"""The hash that ties the committed traffic counters of the gate/up GEMM to its source covers every
file that the kernel is compiled from."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2512_20276_amd", "csrc")


def _includes(path, seen):
    for name in re.findall(r'^#include "([^"]+)"', open(path).read(), flags=re.M):
        p = os.path.join(CSRC, name)
        if "/" not in name and p not in seen:  # the C interface, a folder up, holds no device code
            seen.append(p)
            _includes(p, seen)
    return seen


def test_every_included_file_is_hashed():
    src = os.path.join(CSRC, "af_gemm.hip")
    assert set(bench.KERNEL_SOURCES) == {src, *_includes(src, [])}


def test_the_hash_follows_a_header(tmp_path, monkeypatch):
    before = bench.kernels_sha256()
    copies = []
    for i, p in enumerate(bench.KERNEL_SOURCES):
        copies.append(str(tmp_path / os.path.basename(p)))
        with open(copies[-1], "w") as f:
            f.write(open(p).read() + ("// changed" if "af_epilogue" in p else ""))
    monkeypatch.setattr(bench, "KERNEL_SOURCES", copies)
    assert bench.kernels_sha256() != before


def test_kernel_classes_name_the_streaming_instance():
    for name in ("_ZN2af18gemm_stream_kernelILi5ELi3ELi5EEEvNS_8GemmArgsEi",
                 "void af::gemm_stream_kernel<5, 3, 5>(af::GemmArgs, int)"):
        assert bench._kernel_class(name) == "gemm (streamed, 5 row x 3 column blocks)"
