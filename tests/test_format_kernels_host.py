"""The format and pruning kernels on the CPU: the device code itself, compiled as plain C++ with the compiler's
undefined-behaviour checks (a violation traps), against the oracle bit for bit, and the launch code against
the runtime's limits.  Each call runs in a process of its own, so that a trap fails one test."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from oracle import vnm_oracle as o
from paper_2310_02065_amd import build, inputs

HERE = os.path.dirname(os.path.abspath(__file__))
c, p64 = ctypes, ctypes.c_int64


def clang():
    return os.path.join(os.path.dirname(os.path.realpath(build.hipcc())), "..", "lib", "llvm", "bin", "clang++")


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_kernels") / "libhost.so")
    subprocess.run([clang(), "-x", "c++", "-std=c++20", "-O1", "-fPIC", "-shared",
                    "-fsanitize=undefined", "-fsanitize-trap=all", "-Wno-everything",
                    "-I", os.path.join(HERE, "host_kernels"), "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"),
                    os.path.join(HERE, "host_kernels", "driver.cpp"), "-o", out], check=True)
    return out


def in_child(library, function, *args):
    code = (f"import sys; sys.path[:0] = [{build.ROOT!r}, {HERE!r}]; import test_format_kernels_host as t; "
            f"t.{function}(t.load({library!r}), *{args!r})")
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, f"exit status {res.returncode}\n{res.stdout[-2000:]}{res.stderr[-2000:]}"


def load(path):
    L = c.CDLL(path)
    vp, i = c.c_void_p, c.c_int
    L.host_workspace_bytes.argtypes, L.host_workspace_bytes.restype = [p64, p64, i, i], c.c_size_t
    L.host_launches.restype = L.host_blocks.restype = c.c_uint64
    L.host_compress.argtypes = [vp, p64, vp, p64, p64, p64, i, i, vp, vp]
    L.host_import.argtypes = [vp, vp, vp, p64, p64, i, i, vp, vp]
    L.host_compress_with_slot.argtypes = [vp, p64, vp, p64, p64, p64, i, i, vp, i, vp, vp]
    L.host_import_with_slot.argtypes = [vp, vp, vp, p64, p64, i, i, vp, i, vp, vp]
    L.host_export.argtypes = [p64, p64, i, i, vp, vp, vp, vp]
    L.host_decompress.argtypes = [p64, p64, i, i, vp, vp, p64]
    L.host_prune.argtypes = [vp, p64, p64, p64, i, i, vp, p64, vp, vp]
    return L


def aligned(nbytes, offset=0, fill=0xA5):
    """nbytes of memory `offset` bytes past a 256-byte boundary."""
    raw = np.full(nbytes + 512, fill, dtype=np.uint8)
    start = (-raw.ctypes.data) % 256 + offset
    return raw[start:start + nbytes]


def pitched(a, pitch, offset=0):
    """`a` in rows of `pitch` elements, the first one `offset` bytes past a 256-byte boundary."""
    mem = aligned(a.shape[0] * pitch * a.itemsize, offset).view(a.dtype).reshape(a.shape[0], pitch)
    mem[:, :a.shape[1]] = a
    return mem


def problem(R, K, V, M):
    rng = np.random.default_rng(R + K + V)
    A = (rng.standard_normal((R, K)) * 0.05).astype(np.float16).view(np.uint16)
    mask = np.where(rng.random((R, K)) < 0.2, 0, inputs.gen_mask(R, K, V, M, rng)).astype(np.uint8)
    return A, mask * rng.integers(1, 256, (R, K)).astype(np.uint8)


def exported(L, R, K, V, M, ws):
    G = K // M
    out = (np.zeros((R, G, 2), np.uint16), np.zeros((R // V, G, 4), np.uint16), np.zeros((R, (G + 7) // 8), np.uint32))
    L.host_export(R, K, V, M, ws.ctypes.data, *(x.ctypes.data for x in out))
    return out


def check_compress(L, R, K, V, M, ldm, offset):
    A, mask = problem(R, K, V, M)
    m = pitched(mask, ldm, offset)
    ws, legal = aligned(L.host_workspace_bytes(R, K, V, M)), np.zeros(1, np.uint64)
    assert L.host_compress(A.ctypes.data, K, m.ctypes.data, ldm, R, K, V, M, ws.ctypes.data, legal.ctypes.data) == 0
    assert legal[0] == np.uint64(2**64 - 1)
    for got, want in zip(exported(L, R, K, V, M, ws), o.compress(A, (mask != 0).astype(np.uint8), V, M)):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("R,K,V,M,ldm,offset", [
    (64, 36, 32, 4, 48, 0),          # 16-byte mask loads, and a last word narrower than one of them
    (64, 45, 32, 5, 48, 8),          # 8-byte loads, likewise
    (64, 60, 32, 4, 64, 0),          # a last word that is a whole load and a remainder
    (64, 92, 32, 4, 96, 8),          # the same with 8-byte loads
    (64, 45, 32, 5, 45, 1), (64, 60, 32, 4, 61, 3),   # rows at every alignment, both load widths
    (8192, 45, 8192, 5, 45, 2),      # ... and a block too tall for bits on chip
    (96, 9 * 32, 96, 32, 288, 0), (128, 9 * 33, 128, 33, 297, 1),   # eight rows in flight: three and four a thread
    (64, 9 * 32, 64, 32, 288, 0), (6, 9 * 40, 2, 40, 360, 0),       # two, as threads have fewer
])
def test_compress(library, R, K, V, M, ldm, offset):
    in_child(library, "check_compress", R, K, V, M, ldm, offset)


def at(a, offset):
    """The bytes of `a`, `offset` bytes past a 256-byte boundary."""
    mem = aligned(a.nbytes, offset)
    mem[:] = np.frombuffer(a.tobytes(), np.uint8)
    return mem


def check_import(L, R, K, V, M, *offsets):
    A, mask = problem(R, K, V, M)
    arrays = o.compress(A, (mask != 0).astype(np.uint8), V, M)
    moved = [at(a, off) for a, off in zip(arrays, offsets)]
    ws, legal = aligned(L.host_workspace_bytes(R, K, V, M)), np.zeros(1, np.uint64)
    assert L.host_import(*(m.ctypes.data for m in moved), R, K, V, M, ws.ctypes.data, legal.ctypes.data) == 0
    assert legal[0] == np.uint64(2**64 - 1)
    for got, want in zip(exported(L, R, K, V, M, ws), arrays):
        assert np.array_equal(got, want)
    if V % 32 == 0:
        dense = aligned(R * K * 2).view(np.uint16).reshape(R, K)
        assert L.host_decompress(R, K, V, M, ws.ctypes.data, dense.ctypes.data, K) == 0
        assert np.array_equal(dense, np.where(mask != 0, A, 0))


@pytest.mark.parametrize("R,K,V,M,offsets", [
    (64, 12 * 8, 32, 8, (0, 0, 0)),
    (64, 12 * 8, 32, 8, (2, 2, 4)),  # arrays sliced out of larger ones
    (64, 11 * 7, 32, 7, (6, 6, 8)),  # ... and groups per row that are no multiple of 4
    (9, 11 * 5, 1, 5, (1, 3, 5)),    # any byte
])
def test_import(library, R, K, V, M, offsets):
    in_child(library, "check_import", R, K, V, M, *offsets)


def check_decompress(L, R, K, V, M, lda, offset):
    A, mask = problem(R, K, V, M)
    ws, legal = aligned(L.host_workspace_bytes(R, K, V, M)), np.zeros(1, np.uint64)
    assert L.host_compress(A.ctypes.data, K, mask.ctypes.data, K, R, K, V, M, ws.ctypes.data, legal.ctypes.data) == 0
    dense = pitched(np.full((R, K), 7, np.uint16), lda, offset)
    assert L.host_decompress(R, K, V, M, ws.ctypes.data, dense.ctypes.data, lda) == 0
    assert np.array_equal(dense[:, :K], np.where(mask != 0, A, 0)) and (dense[:, K:] == 0xA5A5).all()


@pytest.mark.parametrize("R,K,V,M,lda,offset", [
    (128, 4, 32, 4, 4, 0), (128, 20, 64, 4, 21, 2),   # one group; five, the last one without its pair
    (128, 268, 128, 4, 272, 0),      # a second chunk of columns, its last piece four wide
    (64, 35, 32, 5, 37, 6),          # three groups under eight columns
    (96, 330, 96, 6, 331, 4), (64, 534, 32, 6, 534, 2), (64, 63, 64, 7, 64, 0),   # two, at M = 6 each offset in the group
    (64, 27, 32, 9, 27, 2), (64, 300, 64, 10, 301, 14),
    (64, 520, 32, 8, 520, 0), (128, 96, 128, 32, 97, 2),   # one group
    (320, 700, 64, 7, 701, 2), (288, 600, 96, 20, 600, 0), (288, 600, 96, 20, 604, 0),   # 30 and 27 workgroups, over XCDs or not
    (64, 160, 32, 10, 160, 0), (64, 75, 64, 5, 80, 0),   # pairs of groups and their ends, rows on 16-byte boundaries
])
def test_decompress(library, R, K, V, M, lda, offset):
    in_child(library, "check_decompress", R, K, V, M, lda, offset)


def check_violations(L, R, K, V, M, places):
    """Legal, then with a whole group kept in each row of `places`, then legal again, in one slot."""
    A, mask = problem(R, K, V, M)
    bad = mask.copy()
    for row, g in places:
        bad[row, g * M:(g + 1) * M] = 1
    status, where = o.check_mask(bad, V, M)
    key = (where[0] * (K // M) + where[1]) << 24 | (status == o.ERR_MASK_ROW and 1 << 23 | where[2] % V)
    ws, one = aligned(L.host_workspace_bytes(R, K, V, M)), np.zeros(1, np.uint64)
    none = 2**64 - 1
    for m, want in ((mask, none), (bad, key), (mask, none), (np.ones_like(mask), 0 if M > 4 else 1 << 23)):
        found, legal = np.zeros(1, np.uint64), np.zeros(2, np.uint64)
        assert L.host_compress_with_slot(A.ctypes.data, K, m.ctypes.data, K, R, K, V, M, ws.ctypes.data, 63, found.ctypes.data,
                                         legal.ctypes.data) == 0
        assert (found[0] != 0) == (want != none) and int(legal[0]) == want and int(legal[1]) == none
        assert L.host_compress(A.ctypes.data, K, m.ctypes.data, K, R, K, V, M, ws.ctypes.data, one.ctypes.data) == 0
        assert int(one[0]) == want
    arrays = o.compress(A, mask, V, M)
    for row, word in ((None, None), (R - 1, arrays[2].shape[1] - 1), (0, 0), (None, None)):
        meta = arrays[2].copy()
        if row is not None:
            meta[row, word] = 0
        found, legal = np.zeros(1, np.uint64), np.zeros(2, np.uint64)
        assert L.host_import_with_slot(arrays[0].ctypes.data, arrays[1].ctypes.data, meta.ctypes.data, R, K, V, M, ws.ctypes.data,
                                       0, found.ctypes.data, legal.ctypes.data) == 0
        assert (found[0] != 0) == (row is not None) == (int(legal[0]) != none) and int(legal[1]) == none


@pytest.mark.parametrize("R,K,V,M,places", [
    (128, 264, 32, 8, ((97, 3), (70, 20), (66, 20), (40, 32))),      # packed copies; the last group of a ragged word
    (64, 130, 1, 5, ((63, 25), (9, 7))),                             # a row to a block, no packed copies
    (128, 64, 64, 4, ((100, 1), (3, 9), (2, 9))),                    # M = 4: only the row rule
])
def test_violations(library, R, K, V, M, places):
    in_child(library, "check_violations", R, K, V, M, places)


def check_decompress_launch(L, R, K, V, M):
    L.host_dry_run(1)
    assert L.host_decompress(R, K, V, M, 0, 0, K) == 0
    assert L.host_blocks() == R // 32 * ((K + 255) // 256)
    if R * K < 2**31:
        assert L.host_launches() == 1


@pytest.mark.parametrize("R,K,V,M", [
    (2**29, 4, 2**14, 4),            # one column chunk per row: as many workgroups as the launch limit and one more
    (2**30 - 2**15, 4, 2**14, 4),    # the tallest such matrix
    (128, 2**31 - 32, 128, 32),      # 2^23 column chunks per row
    (8192, 8192, 64, 8),
])
def test_decompress_launches_within_limits(library, R, K, V, M):
    in_child(library, "check_decompress_launch", R, K, V, M)


def check_prune_launch(L, R, K, V, M):
    L.host_dry_run(1)
    assert L.host_prune(0, K, R, K, V, M, 0, K, 0, 0) == 0
    assert L.host_launches() == 1


@pytest.mark.parametrize("R,K,V,M", [
    (1, 2**31 - 32, 1, 32),          # 128 columns per workgroup would be 2^24 workgroups
    (32, 2**31 - 64, 32, 64),
    (1, 2**31 - 128, 1, 128),        # 2^24 - 1
])
def test_prune_launches_within_limits(library, R, K, V, M):
    in_child(library, "check_prune_launch", R, K, V, M)


def check_prune(L, R, K, V, M, lda, offset):
    A, _ = problem(R, K, V, M)
    a = pitched(A, lda, offset)
    mask = pitched(np.full((R, K), 7, np.uint8), K + 3)
    kept, total = np.zeros(R // V, np.uint64), np.zeros(R // V, np.uint64)
    assert L.host_prune(a.ctypes.data, lda, R, K, V, M, mask.ctypes.data, K + 3, kept.ctypes.data, total.ctypes.data) == 0
    want, want_kept, want_total = o.prune(A, V, M)
    assert np.array_equal(mask[:, :K], want) and (mask[:, K:] == 0xA5).all()
    assert int(kept.sum()) == want_kept and int(total.sum()) == want_total


@pytest.mark.parametrize("R,K,V,M,lda,offset", [
    (64, 160, 32, 10, 160, 0),
    (64, 170, 32, 10, 171, 2),       # rows at every 2-byte boundary, two columns left over
    (64, 4, 32, 4, 5, 6),            # rows narrower than one load
    (6, 210, 3, 7, 213, 14),
    (4, 1100, 2, 100, 1104, 0),      # few rows: a tile of 1000 columns, and one group
    (32, 1304, 32, 8, 1304, 0), (64, 816, 64, 16, 817, 2),   # tiles of 512 and 256 columns, and a narrower last one
    (48, 1120, 48, 10, 1120, 0), (56, 560, 56, 7, 560, 0),   # 280 columns, and 168
    (96, 500, 32, 100, 501, 2), (64, 455, 64, 65, 455, 0),   # groups above 64 columns, a group's mask in words of 4 bytes and in bytes
    (288, 504, 32, 72, 504, 0), (32, 384, 32, 128, 384, 0),   # ... of 8, and of 4 as the mask's rows are on no boundary
    (96, 612, 32, 204, 613, 2), (24, 1250, 24, 250, 1250, 0),   # mask pieces over two groups, the last of a row shorter
    (288, 408, 32, 204, 408, 0), (32, 1024, 32, 256, 1024, 0),   # ... workgroups over XCDs, and some left
    (640, 54, 640, 6, 55, 2),        # a tile of 24 columns
    (1024, 128, 1024, 64, 128, 0), (1024, 64, 1024, 64, 67, 6),   # too tall for a tile: the general kernel, wide loads and not
])
def test_prune(library, R, K, V, M, lda, offset):
    in_child(library, "check_prune", R, K, V, M, lda, offset)
