"""bench.py attaches committed counters to a kernel only while their hash is that
of its sources: the hash has to cover every source that the kernel is made of."""
import os
import re

import pytest

import bench


def _sources(name, seen):
    path = os.path.join(bench.CSRC, name)
    if name in seen or not os.path.exists(path):   # the C header holds no device code
        return seen
    seen.add(name)
    with open(path) as fh:
        for inc in re.findall(r'^#include "([^"]+)"', fh.read(), re.M):
            _sources(inc, seen)
    return seen


@pytest.mark.parametrize("hash_of,main", [(bench.bgk_src_hash, "lbm_kernels.hip"),
                                          (bench.simple_src_hash, "simple_kernels.hip"),
                                          (bench.gnn_src_hash, "gnn_kernels.hip")])
def test_hash_covers_the_sources_of_its_kernel(monkeypatch, hash_of, main):
    whole, real = hash_of(), bench._read
    need = _sources(main, set())
    assert main in need and len(need) > 1
    for name in need - {main}:
        monkeypatch.setattr(bench, "_read",
                            lambda n, name=name: real(n) + (b" " if n == name else b""))
        assert hash_of() != whole, f"{name} is not covered"
