"""The stored counters of bench.py count only while the kernel's sources are those
they were taken with: the hash covers kernels.hip and every header of the
library that it includes."""

import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_sources", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _included(path, seen):
    seen.add(os.path.realpath(path))
    for name in re.findall(r'#include\s+"([^"]+)"', open(path).read()):
        sub = os.path.realpath(os.path.join(os.path.dirname(path), name))
        if os.path.exists(sub) and sub not in seen:
            _included(sub, seen)
    return seen


def test_hash_covers_the_device_code(tmp_path):
    b = _bench()
    csrc = os.path.join(ROOT, "paper_1402_3545_amd", "csrc")
    want = {p for p in _included(os.path.join(csrc, "kernels.hip"), set())
            if os.path.dirname(p) == os.path.realpath(csrc)}
    assert {os.path.realpath(p) for p in b.KERNEL_SOURCES} == want
    # a change in any of them changes the hash
    before = b.source_sha256()
    for k, path in enumerate(b.KERNEL_SOURCES):
        edited = tmp_path / os.path.basename(path)
        edited.write_bytes(open(path, "rb").read() + b"\n")
        b.KERNEL_SOURCES[k], keep = str(edited), path
        assert b.source_sha256() != before
        b.KERNEL_SOURCES[k] = keep
    assert b.source_sha256() == before
