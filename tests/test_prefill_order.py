"""The workgroup order of the prefill attention (csrc/prefill_order.h, compiled for the host): every block of query
positions exactly once, and each KV head's blocks spread over the XCDs and their shader engines."""
import ctypes
import os
import random
import shutil
import subprocess
from types import SimpleNamespace

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    so = str(tmp_path_factory.mktemp("order") / "prefill_order.so")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared", "-I",
                        os.path.join(ROOT, "paper_2511_03092_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "prefill_order.cpp"), "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(so)
    lib.prefill_fits.argtypes, lib.prefill_fits.restype = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    return lib


def _order(lib, *call):
    o = (ctypes.c_longlong * 6)()
    lib.prefill_order_of(*call, o)
    return SimpleNamespace(**dict(zip(("waves", "P", "n_qblocks", "groups", "whole", "grid"), o)))


def _blocks(lib, *call):
    o = _order(lib, *call)
    g, b = np.empty(o.grid, np.int32), np.empty(o.grid, np.int32)
    p = ctypes.POINTER(ctypes.c_int)
    lib.prefill_blocks_of(*call, g.ctypes.data_as(p), b.ctypes.data_as(p))
    return o, g, b


def _calls():
    """(n_seq, KV heads, G, d, max_len): edges of the block size and of the groups on 8 XCDs, then random ones."""
    for hkv in (1, 3, 7, 8, 9, 12, 16):
        for n in (1, 2, 5):
            for length in (1, 15, 16, 17, 129, 1000):
                yield n, hkv, 4, 128, length
    rng = random.Random(3)
    for _ in range(300):
        yield (rng.choice([1, 2, 3, 4, 8, 13, 32]), rng.randint(1, 20), rng.choice([1, 2, 4, 8, 16]),
               rng.choice([64, 128]), int(round(2 ** rng.uniform(0, 13))))


def test_every_block_once(lib):
    for call in _calls():
        o, g, b = _blocks(lib, *call)
        assert o.P * (o.n_qblocks - 1) < call[4] <= o.P * o.n_qblocks and o.P * call[2] == 32 * o.waves, call
        assert o.grid == o.groups * o.n_qblocks, call
        assert g.min() >= 0 and g.max() < o.groups and b.min() >= 0 and b.max() < o.n_qblocks, call
        assert len(np.unique(g.astype(np.int64) * o.n_qblocks + b)) == o.grid, call


def test_a_group_goes_round_the_xcds(lib):
    """A spread group's blocks: each of any 8 * turn consecutive ones' XCDs equally often."""
    for call in _calls():
        o, g, b = _blocks(lib, *call)
        n_whole = o.whole * o.n_qblocks
        at = np.empty((o.groups, o.n_qblocks), np.int64)
        at[g, b] = np.arange(o.grid)
        for row in at[o.whole:]:
            counts = np.bincount(row % 8, minlength=8)
            assert counts.max() - counts.min() <= max(2, o.n_qblocks // 32), (call, counts)
        assert n_whole == 0 or (at[:o.whole] % 8 == np.arange(o.whole)[:, None] % 8).all(), call


@pytest.mark.parametrize("n_seq,n_kv_heads", [(8, 4), (16, 2), (32, 1), (16, 4), (24, 4), (32, 4)])
def test_a_group_goes_round_the_engines(lib, n_seq, n_kv_heads):
    """Workgroup i runs on XCD i % 8 and, there, on shader engine i / 8 % 4: of any 8 consecutive blocks of a group each
    engine has one to three, so no engine has the long sequences (changing places by one XCD a block, an engine kept a
    group for 8 blocks)."""
    o, g, b = _blocks(lib, n_seq, n_kv_heads, 8, 128, 1024)
    assert o.whole == 0 and o.groups % 32 == 0 and o.n_qblocks >= 32
    at = np.empty((o.groups, o.n_qblocks), np.int64)
    at[g, b] = np.arange(o.grid)
    engine = at // 8 % 4
    for k in range(o.n_qblocks - 7):
        counts = np.stack([(engine[:, k:k + 8] == e).sum(1) for e in range(4)])
        assert counts.min() >= 1 and counts.max() <= 3, (k, counts)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 8, 16])
def test_largest_accepted_grids(lib, G, d):
    """The longest prompts that a call may have: its grid, in whole numbers, is within the launch limit (a 64-wide one
    in workgroups of half the positions would have twice that)."""
    positions = 256 // G
    for n_seq, n_kv_heads in ((1, 513), (8, 1024), (4096, 15), (65535, 1)):
        groups = n_seq * n_kv_heads
        longest = min(0x7fffffff // (-(-groups // 8) * 8) * positions, 1 << 28)
        assert lib.prefill_fits(groups, G, longest)
        assert longest == 1 << 28 or not lib.prefill_fits(groups, G, longest + 1)
        o = _order(lib, n_seq, n_kv_heads, G, d, longest)
        assert o.grid == groups * -(-longest // o.P) <= 0x7fffffff and o.P * G == 32 * o.waves, (groups, longest)


@pytest.mark.parametrize("groups", [1, 8, 16, 17, 31, 32, 48, 63])
def test_rescore_groups_start_on_all_engines(lib, groups):
    """The first workgroups of the groups' fp64 re-scores, which have the work of short latent prompts, are spread over
    the 8 XCDs and the four shader engines of each; from 64 groups on, and for narrow keys, 16 workgroups a group."""
    n = lib.band_workgroups_of(576, groups)
    first = [g * n for g in range(groups)]
    places = {(i % 8, i // 8 % 4) for i in first}
    assert len(places) == min(groups, 32)
    assert lib.band_workgroups_of(576, 64) == lib.band_workgroups_of(576, 1000) == 16
    assert lib.band_workgroups_of(64, groups) == lib.band_workgroups_of(128, groups) == 16
