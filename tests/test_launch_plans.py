"""The launch plans' arithmetic (csrc/ckv_plan.h), compiled for the host."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2508_02401_amd import build as B
from tests.test_abi_cpu import _resource_usage

SHIM = r"""
#include "ckv_plan.h"
extern "C" {
int64_t chunk_len(int64_t target, int64_t n_kv, int32_t cnt, const int64_t* n) {
  return ckv::decode_chunk_len(target, n_kv, cnt, n);
}
int per_cu(int f32, int d, int rows) { return ckv::decode_wgs_per_cu(f32 != 0, d, rows); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + B.CSRC,
                    str(src), "-o", str(lib)], check=True)
    so = ctypes.CDLL(str(lib))
    so.chunk_len.restype = ctypes.c_int64
    so.chunk_len.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32,
                             ctypes.POINTER(ctypes.c_int64)]
    return so


def _chunk(plan, target, n_kv, lens):
    return plan.chunk_len(target, n_kv, len(lens), (ctypes.c_int64 * len(lens))(*lens))


def _batches():
    yield 32, [131072] + [1024] * 16
    yield 32, [1024] * 16 + [131072]
    yield 8, [131072] + [1024] * 23
    yield 32, [4096] * 24
    yield 4, [8192, 24576, 65536, 98304]
    yield 8, [97, 128, 251, 256, 300, 385, 512, 513, 640, 777, 1024, 1024, 1333, 1536, 2047, 2048]
    yield 1, [1]
    yield 128, [(1 << 31) - 1] * 24
    rng = random.Random(11)
    for _ in range(400):
        top = rng.choice([200, 5000, 131072, 1 << 30])
        yield rng.choice([1, 2, 4, 7, 8, 16, 32, 64, 600]), [
            int(top ** rng.random()) for _ in range(rng.randint(1, 24))]


@pytest.mark.parametrize("target", [256, 512])
def test_decode_chunks_are_balanced_and_one_round_where_they_can_be(plan, target):
    for n_kv, lens in _batches():
        c = _chunk(plan, target, n_kv, lens)
        assert c % 32 == 0 and 128 <= c <= 1 << 31, (n_kv, lens, c)
        even = max(128, -(-(-(-sum(lens) * n_kv // target)) // 32) * 32)
        wgs = sum(-(-n // c) for n in lens) * n_kv
        units = len(lens) * n_kv
        # no workgroup walks more than twice the even share of the keys
        assert min(c, max(lens)) <= 2 * even, (n_kv, lens, c)
        # every cache and head has at most one workgroup past its even share
        assert wgs <= target + units, (n_kv, lens, c)
        # one round whenever twice the even share is surely enough for it
        if units <= target // 2 - 16 and even > 1024:
            assert wgs <= target, (n_kv, lens, c)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dt", [0, 1, 2])
def test_decode_is_cut_for_workgroups_that_the_kernels_admit(plan, dt, d):
    # workgroups of 4 waves, one on each SIMD: 512 registers a lane to share out
    # in eights, and 160 KB of LDS a CU
    usage = _resource_usage()
    for rows in (1, 32, 33, 64, 65, 128):
        kernel = ("13decode_kernelILi%dELi%dELi%dE" % (dt, d, 1 if rows <= 32 else 2) if rows <= 64 else
                  "decode_rows_kernel_%sILi%dELi%dE" % ("f32" if dt == 2 else "16", dt, d))
        u = [v for k, v in usage.items() if kernel in k]
        assert len(u) == 1, kernel
        admit = min(512 // (-(-u[0]["regs"] // 8) * 8), 160 * 1024 // u[0]["lds"], 2)
        # cut for one workgroup of longer chunks although two fit: measured faster
        longer = d == 64 and (dt == 2 and rows <= 32 or dt != 2 and 32 < rows <= 64)
        assert plan.per_cu(dt == 2, d, rows) == (1 if longer else admit), (kernel, u[0])
