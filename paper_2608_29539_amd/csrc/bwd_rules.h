// bwd_rules.h -- which rows a wave of bwd_dkv_kernel computes, masks and
// skips.  Apart from the kernel so that the same functions also compile for the
// CPU, where a test checks them against the pairs themselves (constexpr
// functions run on both sides).
#pragma once

namespace logo {

constexpr int kTileRows = 64;            // rows of a staged tile (keys or queries)
constexpr int kWaveKeys = 32;            // keys of a dK / dV wave
constexpr int kKeysPerWg = 4 * kWaveKeys;

constexpr int lesser(long long a, long long b) { return (int)(a < b ? a : b); }
constexpr int greater(int a, int b) { return a > b ? a : b; }

// Does the row at position qpos see the key at position key (window w, which
// may be the largest int, of the local branch; both positions are of one
// sequence)?
template <bool kLocal>
constexpr bool row_sees_key(int qpos, int key, int w) {
    return (key <= qpos) & (!kLocal | (qpos - key < w));
}

// End of the local branch's rows k0 .. that can see a key of the workgroup's
// block k0 .. k0 + kKeysPerWg - 1 of a sequence of T tokens.
constexpr int local_row_end(int T, int k0, int w) {
    return lesser(T, (long long)k0 + kKeysPerWg - 1 + w);
}

// The tiles first .. last of the block's nblk tiles of rows that the wave with
// the keys j0 .. j0 + 31 computes (first = nblk: none; every other one is only
// staged for the other waves), and among them the ones that need no mask,
// full .. full_end - 1: 64 rows that all see all of the wave's keys.
struct DkvTiles {
    int first, last, full, full_end;
};

// n_rows rows at the ascending positions pos(0) .. pos(n_rows - 1) (local: k0,
// k0 + 1, ...; global: the selected ones from k0 on).
template <bool kLocal, class Pos>
constexpr DkvTiles dkv_tiles(int n_rows, Pos pos, int T, int k0, int j0, int w) {
    const int nblk = (n_rows + kTileRows - 1) / kTileRows;
    DkvTiles t{0, nblk - 1, 0, n_rows / kTileRows};
    if (j0 >= T) {
        t.first = nblk;
        return t;
    }
    while (t.first < nblk && pos(lesser(t.first * kTileRows + kTileRows, n_rows) - 1) < j0)
        t.first++;
    t.full = t.first;
    while (t.full < nblk && pos(t.full * kTileRows) < j0 + kWaveKeys - 1)
        t.full++;
    if (kLocal) {
        // the last row that sees the wave's last key, and the rows from k0 on
        // that see its first one
        const long long jmax = lesser(j0 + kWaveKeys - 1, T - 1);
        t.last = lesser(t.last, (jmax + w - 1 - k0) / kTileRows);
        t.full_end = lesser(t.full_end, ((long long)j0 + w - k0) / kTileRows);
    }
    if (j0 + kWaveKeys - 1 >= T)
        t.full_end = 0;
    t.full_end = greater(t.full, t.full_end);
    return t;
}

}  // namespace logo
