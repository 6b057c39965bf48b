"""Index rules of the kernels that can be checked without a GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pk():
    import paper_2608_29539_amd as pk
    if not os.path.exists(pk.library_path()):
        from paper_2608_29539_amd.build import build_library
        build_library()
    return pk


@pytest.mark.parametrize("B,max_seqlen,hq,hkv,d,win,keys", [
    # one cache: up to 32 chunks of each length
    (1, 200, 8, 2, 128, 64, 128), (1, 4096, 8, 2, 128, 512, 128),
    (1, 4097, 8, 2, 128, 512, 256), (1, 8192, 8, 2, 128, 512, 256), (1, 8193, 8, 2, 128, 512, 512),
    (1, 65536, 8, 2, 128, 512, 512), (1, 65537, 8, 2, 128, 512, 544),
    # 1024 work items with 512 keys, with 256; heads per item 4, 2 and 1
    (64, 300, 16, 8, 64, 200, 512), (63, 1024, 16, 4, 64, 512, 256), (16, 600, 16, 16, 64, 200, 256),
    (40, 300, 16, 8, 64, 200, 128), (16, 2047, 6, 2, 64, 256, 128),
    # a chunk of more than half of the longest cache, above and up to 512 items
    (43, 200, 16, 4, 128, 512, 512), (32, 200, 16, 4, 128, 512, 128), (65, 255, 8, 2, 64, 512, 512),
    (64, 255, 8, 2, 64, 512, 128), (65, 256, 8, 2, 64, 512, 128),
    (32, 300, 32, 8, 128, 512, 512), (40, 300, 32, 8, 64, 512, 512), (16, 300, 16, 16, 128, 512, 512),
    (16, 300, 32, 8, 128, 512, 128), (100, 150, 8, 4, 128, 128, 512), (1, 511, 8, 2, 64, 511, 128),
])
def test_decode_chunks(pk, B, max_seqlen, hq, hkv, d, win, keys):
    """Keys per chunk of a decoding step, from the workspace that the library
    asks for: its partial results are one slot per work item and branch."""
    import paper_2608_29539_amd.binding as b
    cu = np.zeros(B + 1, np.int32)

    def ws(longest):
        p = b._Problem(B, B, longest, cu.ctypes.data_as(ctypes.c_void_p), None, hq, hkv, d, win,
                       0.0)
        return pk.library().logo_workspace_bytes(ctypes.byref(p), pk.LOGO_ENTRY_DECODE, 0)

    g = hq // hkv
    gh = 4 if g % 4 == 0 else 2 if g % 2 == 0 else 1
    slots = B * (hq // gh)

    def partials(longest, kc):
        n = [-(-min(longest, w) // kc) * slots for w in (win, longest)]
        return sum(-(-4 * gh * (d + 2) * i // 256) * 256 for i in n)

    # (a step of one-token caches has one chunk per branch)
    assert ws(max_seqlen) - ws(1) == partials(max_seqlen, keys) - partials(1, keys)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """The rules of csrc/bwd_rules.h, which bwd_dkv_kernel calls, on the CPU."""
    so = str(tmp_path_factory.mktemp("rules") / "rules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared",
                    "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-static-libubsan", "-I", os.path.join(ROOT, "paper_2608_29539_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "dkv_tiles.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


BIG = 2**31 - 1


def _check_tiles(rules, local, pos, T, k0, w):
    """Every tile of 64 rows against its pairs: the tiles that a wave leaves out
    have none, those without a mask have all 64 x 32, and the mask of the others
    is the definition."""
    pos = np.ascontiguousarray(pos, np.int32)
    nblk = -(-pos.size // 64)
    for wave in range(4):
        j0 = k0 + wave * 32
        out = (ctypes.c_int * 4)()
        rules.dkv_tiles(int(local), pos.ctypes.data_as(ctypes.c_void_p), pos.size, T, k0, wave, w,
                        out)
        first, last, full, full_end = out
        keys = np.arange(j0, min(j0 + 32, T), dtype=np.int64)[None, :]
        for q in range(nblk):
            rows = pos[q * 64:q * 64 + 64].astype(np.int64)[:, None]
            sees = (keys <= rows) & ((rows - keys < w) | (not local))
            tag = (local, T, w, k0, wave, q, list(out))
            assert not sees.any() or first <= q <= last, tag
            if first < nblk and full <= q < full_end:
                assert sees.shape == (64, 32) and sees.all() and first <= q <= last, tag
        if first < nblk:
            # (the kernel's loops run from the last tile to the first)
            assert 0 <= first <= full <= full_end <= last + 1 <= nblk, (local, T, w, k0, wave)


@pytest.mark.parametrize("T,w,k0", [
    (1, 1, 0), (300, 1, 128), (300, 64, 128), (700, 257, 256), (513, 5000, 384), (129, 16, 128),
    (640, 128, 0), (1000, 100, 896), (1000, BIG, 0), (257, BIG, 256), (200, BIG - 64, 128),
    (900, 33, 640), (127, 127, 0), (2000, 1000, 128), (700, 127, 128), (2000, 1087, 640),
])
def test_dkv_tile_ranges_local(rules, T, w, k0):
    end = rules.local_row_end(T, k0, w)
    # the rows past the end see none of the block's keys, the last one does
    assert end == max(r for r in range(k0, T) if r - min(k0 + 127, T - 1, r) < w) + 1
    _check_tiles(rules, True, np.arange(k0, end), T, k0, w)


@pytest.mark.parametrize("seed", range(24))
def test_dkv_tile_ranges_global(rules, seed):
    """Selected rows from the block on: none, few, bursts, nearly all."""
    rng = np.random.default_rng(8800 + seed)
    T = int(rng.choice([1, 31, 128, 129, 500, 1500, 4000]))
    k0 = 128 * int(rng.integers(0, -(-T // 128)))
    p = float(rng.choice([0.0, 0.02, 0.3, 0.9, 1.0]))
    pos = k0 + np.nonzero(rng.random(T - k0) < p)[0]
    _check_tiles(rules, False, pos, T, k0, 1)


def test_dkv_mask(rules):
    for w in (1, 2, 63, 1000, BIG):
        for q, k in [(0, 0), (5, 5), (5, 6), (70, 7), (70, 8), (1000, 0), (BIG, 0), (BIG, 1),
                     (BIG - 1, BIG), (0, BIG)]:
            assert rules.row_sees_key(0, q, k, w) == (k <= q), (q, k, w)
            assert rules.row_sees_key(1, q, k, w) == (k <= q and q - k < w), (q, k, w)
