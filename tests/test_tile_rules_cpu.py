"""Index rules of the kernels that can be checked without a GPU."""
import ctypes
import os

import numpy as np
import pytest


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


def test_dkv_tile_ranges():
    """The ranges of 64-row tiles that a 32-key wave computes (qf .. ql) and of
    those without a mask (qa .. qb - 1), as bwd_dkv_kernel forms them for the
    local branch, against the pairs themselves."""
    for T, w, k0 in [(1, 1, 0), (300, 1, 128), (300, 64, 128), (700, 257, 256), (513, 5000, 384),
                     (129, 16, 128), (640, 128, 0), (1000, 100, 896)]:
        r_end = min(T, k0 + 127 + w)
        nblk = -(-(r_end - k0) // 64)
        for wave in range(4):
            j0 = k0 + wave * 32
            qf, ql, qa, qb = 0, nblk - 1, 0, (r_end - k0) // 64
            if j0 >= T:
                continue
            while qf < nblk and min(k0 + qf * 64 + 64, r_end) - 1 < j0:
                qf += 1
            qa = qf
            while qa < nblk and k0 + qa * 64 < j0 + 31:
                qa += 1
            jmax = min(j0 + 31, T - 1)
            ql = min(ql, (jmax + w - 1 - k0) // 64)
            qb = min(qb, (j0 + w - k0) // 64)
            if j0 + 31 >= T:
                qb = 0
            qb = max(qa, min(qb, ql + 1))
            for q in range(nblk):
                rows = np.arange(k0 + q * 64, min(k0 + q * 64 + 64, r_end))[:, None]
                keys = np.arange(j0, jmax + 1)[None, :]
                sees = (keys <= rows) & (rows < keys + w)
                assert not sees.any() or qf <= q <= ql, (T, w, k0, wave, q)
                if qa <= q < qb:
                    assert rows.size == 64 and keys.size == 32 and sees.all(), (T, w, k0, wave, q)
