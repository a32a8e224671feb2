"""The launch plans' arithmetic (csrc/ckv_plan.h), compiled for the host."""
import ctypes
import os
import random
import subprocess

import pytest
import torch

import paper_2508_02401_amd as ckv
from paper_2508_02401_amd import build as B
from tests.test_abi_cpu import _resource_usage

SHIM = r"""
#include "ckv_plan.h"
extern "C" {
int64_t chunk_len(int64_t target, int64_t n_kv, int32_t cnt, const int64_t* n) {
  return ckv::decode_chunk_len(target, n_kv, cnt, n);
}
int64_t deal(int64_t cus, int32_t n, int32_t n_sg, int32_t heads, const int64_t* rows, int32_t* first,
             int32_t* same) {
  ckv::UnitParts p;
  const int64_t most = ckv::deal_unit_parts(cus, n, n_sg, heads, rows, p);
  for (int32_t s = 0; s <= n; ++s) first[s] = p.first[s];
  *same = p.same;
  return most;
}
int64_t part_round(int64_t cus, int64_t rows, int64_t scored) {
  return ckv::part_round(cus, rows, scored);
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
    so.part_round.restype = ctypes.c_int64
    so.part_round.argtypes = [ctypes.c_int64] * 3
    so.deal.restype = ctypes.c_int64
    so.deal.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.POINTER(ctypes.c_int64),
                        ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
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


# ---- parts of selection units ------------------------------------------------
def _layers():
    yield 8, [8192] + [128] * 15
    yield 8, [16384] + [128] * 15
    yield 16, [4096] + [128] * 15
    yield 64, [512] * 16
    yield 1, [1]
    yield 8, [2048]
    yield 3, [17, 1, 16]
    rng = random.Random(7)
    for _ in range(400):
        yield rng.choice([1, 2, 3, 4, 8, 16, 32, 64]), [
            int(rng.choice([40, 3000, 65536, 1 << 30]) ** rng.random()) for _ in range(rng.randint(1, 16))]


def _deal(plan, n_sg, heads, rows):
    n = len(rows)
    first, same = (ctypes.c_int32 * (n + 1))(), ctypes.c_int32()
    most = plan.deal(256, n, n_sg, heads, (ctypes.c_int64 * n)(*rows), first, ctypes.byref(same))
    assert first[0] == 0 and all((b - a) % n_sg == 0 for a, b in zip(first, first[1:]))
    parts = [(b - a) // n_sg for a, b in zip(first, first[1:])]
    assert same.value == (parts[0] if len(set(parts)) == 1 else 0)
    return most, parts


def test_unit_parts_are_one_round_dealt_out_by_rows(plan):
    for n_sg, rows in _layers():
        units = len(rows) * n_sg
        most, parts = _deal(plan, n_sg, 1, rows)
        assert min(parts) >= 1 and sum(parts) * n_sg <= max(256, units), (n_sg, rows, parts)
        assert most == max(-(-r // p) for r, p in zip(rows, parts))
        assert all(p == 1 or r // p >= 16 for r, p in zip(rows, parts)), (n_sg, rows, parts)
        # the workgroups past one per unit are shared out by rows
        even = sum(rows) * n_sg / max(256 - units, 1)
        assert most <= max(31, even + 1) or units >= 256, (n_sg, rows, parts)
        if len(set(rows)) == 1 and units <= 256 and rows[0] >= 16 * 256:
            assert parts[0] == 256 // units


def test_unit_parts_of_a_shared_selection_keep_to_one_head(plan):
    for heads, rows in _layers():
        most, parts = _deal(plan, 1, heads, rows)
        assert sum(parts) <= 256
        for r, p in zip(rows, parts):
            assert p <= heads or p % heads == 0, (heads, rows, parts)
            assert p == 1 or r * heads // p >= 16
        assert most == max(-(-r * heads // p) for r, p in zip(rows, parts))


def test_unit_parts_leave_half_the_cus_unless_rows_are_many(plan):
    # a part's LDS leaves no room for another layer's K-pass workgroup on its CU
    usage = _resource_usage()
    lds = {k: u["lds"] for k, u in usage.items()}
    parts = max(v for k, v in lds.items() if "select_parts_kernel" in k)
    kpass = min(v for k, v in lds.items() if "rowstats_kernel" in k or "score_kernel" in k)
    assert parts + kpass > 160 * 1024
    assert plan.part_round(256, 1, 8192) == plan.part_round(256, 8 * 4096, 65536) == 128
    # many rows to copy, or short prompts, whose K passes leave CUs free
    assert plan.part_round(256, 8 * 4096 + 1, 65536) == plan.part_round(256, 1, 8191) == 256


# ---- decode workspace sizes: bounds for smaller calls too ------------------
DTYPES = {0: torch.bfloat16, 1: torch.float16, 2: torch.float32}
SHAPES = [(0, 32, 8, 128), (2, 32, 8, 128), (1, 16, 2, 64), (2, 16, 2, 64), (0, 32, 32, 128), (0, 7, 1, 64)]


def _seq(T, n, d):
    """A prompt whose addresses are never touched: only its sizes are read."""
    s = ckv.ckv_decode_seq()
    s.q, s.q_stride_t, s.q_stride_h, s.T, s.out = 1 << 20, 1 << 16, d, T, 1 << 20
    c = s.cache
    c.k, c.v, c.stride_head, c.stride_tok, c.n = 1 << 20, 1 << 20, n * d, d, n
    return s


def _need(plan, dt, H, n_kv, d, prompts):
    """Bytes of partials that a batch of (T, n) uses, in one launch."""
    G = H // n_kv
    rows = max(T for T, _ in prompts) * G
    c = _chunk(plan, 256 * plan.per_cu(dt == 2, d, rows), n_kv, [n for _, n in prompts])
    up = lambda x: -(-x // 256) * 256
    return sum(up(n_kv * -(-n // c) * T * G * (d + 2) * 4) for T, n in prompts)


@pytest.mark.parametrize("dt,H,n_kv,d", SHAPES)
def test_decode_workspace_grows_with_tokens_and_cache(plan, dt, H, n_kv, d):
    desc = ckv.attn_desc(H, n_kv, d, DTYPES[dt])
    lens = [1, 31, 128, 129, 700, 8192, 8193, 20000, 65536, 65537, 131072, 1000003]
    tokens = [T for T in list(range(1, 19)) + [31, 32, 64, 128] if T * H // n_kv <= 128]
    size = [[ckv.ckv_decode_workspace_bytes(desc, T, n) for n in lens] for T in tokens]
    err = [[ckv.ckv_layer_error_workspace_bytes(desc, T, n, max(n // 7, 1), 512) for n in lens]
           for T in tokens]
    for a in (size, err):
        for row in a:
            assert row == sorted(row)
        for col in zip(*a):
            assert list(col) == sorted(col)
    for T, row in zip(tokens, size):
        for n, got in zip(lens, row):
            assert got >= _need(plan, dt, H, n_kv, d, [(T, n)]), (T, n)


@pytest.mark.parametrize("dt,H,n_kv,d", SHAPES)
def test_decode_batch_workspace_holds_for_smaller_prompts(plan, dt, H, n_kv, d):
    desc = ckv.attn_desc(H, n_kv, d, DTYPES[dt])
    rng = random.Random(H + dt)
    few = lambda T: T * H // n_kv <= 64
    for _ in range(60):
        cnt = rng.choice([1, 2, 5, 24])
        top = 128 * n_kv // H
        big = [(rng.randint(1, top), int(200000 ** rng.random())) for _ in range(cnt)]
        size = ckv.ckv_decode_batch_workspace_bytes(desc, [_seq(T, n, d) for T, n in big])
        for _ in range(20):
            small = [(rng.randint(1, T), rng.randint(1, n)) for T, n in big]
            assert ckv.ckv_decode_batch_workspace_bytes(
                desc, [_seq(T, n, d) for T, n in small]) <= size, (big, small)
            # together, or the prompts of few rows apart
            a, b = [p for p in small if few(p[0])], [p for p in small if not few(p[0])]
            assert _need(plan, dt, H, n_kv, d, small) <= size
            assert sum(_need(plan, dt, H, n_kv, d, x) for x in (a, b) if x) <= size, (big, small)
