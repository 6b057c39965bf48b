"""Index rules of the kernels that can be checked without a GPU."""
import numpy as np


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
