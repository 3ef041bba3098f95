"""CPU checks of the benchmark's measurement aids: the stamp buffer covers every workgroup of the launch it is given to."""
import ctypes
import os
import subprocess

import pytest

import bench
from paper_2510_12747_amd import binding as B
from paper_2510_12747_amd import build as lib_build


@pytest.fixture(scope="module")
def aids():
    if not os.path.exists(os.path.join(bench.ROOT, "libbench_probe.so")):
        lib_build.build_bench_aids()
    return bench.Aids().lib


@pytest.fixture(scope="module")
def fill(tmp_path_factory):
    """Marks a cache handle full, as appends on a GPU would leave it (the count of visible groups is host state)."""
    tmp = tmp_path_factory.mktemp("fill")
    src, lib = tmp / "fill.hip", tmp / "fill.so"
    src.write_text('#include "lcsa_cache_handle.h"\nextern "C" void fill(lcsa_cache *c) { c->kc.valid = c->kg.cap; }\n')
    subprocess.run(["/opt/rocm/bin/hipcc", *lib_build.FLAGS, "-I", lib_build.CSRC, "-o", str(lib), str(src)], check=True, capture_output=True)
    return ctypes.CDLL(str(lib)).fill


# heads, grid, top-k -> work items on the 256 compute units, and the workgroups the launch must have (a multiple of 8)
@pytest.mark.parametrize("heads,grid,topk,items,workgroups", [
    (12, (24, 44), 16, 216, 216),         # one item per workgroup, split
    (12, (24, 44), 1, 216, 216),          # one item per workgroup, one group idle
    (16, (24, 44), 16, 288, 144),         # pairs
    (12, (48, 64), 32, 576, 576),         # three rounds of split items
    (12, (48, 64), 4, 576, 288),          # the same with rows too short to split
    (12, (48, 88), 32, 864, 432),
    (3, (21, 37), 16, 54, 56),
])
def test_a_stamp_buffer_covers_the_launch_or_is_refused(aids, fill, heads, grid, topk, items, workgroups):
    g = B.Geom(heads, 128, *grid, 8, 16, 2, 6, -1, -1, topk)
    assert g.heads * g.n_qb == items
    L, gc, cache, form = B.lib(), g.c(), ctypes.c_void_p(), ctypes.c_int32()
    fake = ctypes.c_void_p(1 << 20)       # never dereferenced on the host
    assert L.lcsa_cache_init(ctypes.byref(cache), ctypes.byref(gc), fake, B.lcsa_cache_device_bytes(g)) == 0
    timed = lambda rows: aids.bench_attn_timed(ctypes.byref(gc), fake, 1536, 128, cache, fake, fake, fake, 1536, 128, 0.0, fake, rows, None)
    assert timed(1 << 20) == -1           # an empty cache
    fill(cache)
    n = aids.bench_attn_workgroups(ctypes.byref(gc), cache, ctypes.byref(form))
    assert n == workgroups
    assert timed(n - 1) == -1 and timed(0) == -1      # refused before anything is launched
    L.lcsa_cache_free(cache)
