// C entry points to the tile rules of bwd_dkv_kernel (bwd_rules.h), compiled
// for the CPU by tests/test_tile_rules_cpu.py.
#include "bwd_rules.h"

namespace {

template <bool kLocal>
void tiles(const int *pos, int n_rows, int T, int k0, int wave, int w, int out[4]) {
    const logo::DkvTiles t = logo::dkv_tiles<kLocal>(
        n_rows, [&](int i) { return pos[i]; }, T, k0, k0 + wave * logo::kWaveKeys, w);
    out[0] = t.first;
    out[1] = t.last;
    out[2] = t.full;
    out[3] = t.full_end;
}

}  // namespace

extern "C" {

int local_row_end(int T, int k0, int w) { return logo::local_row_end(T, k0, w); }

int row_sees_key(int local, int qpos, int key, int w) {
    return local ? logo::row_sees_key<true>(qpos, key, w) : logo::row_sees_key<false>(qpos, key, w);
}

void dkv_tiles(int local, const int *pos, int n_rows, int T, int k0, int wave, int w, int out[4]) {
    if (local)
        tiles<true>(pos, n_rows, T, k0, wave, w, out);
    else
        tiles<false>(pos, n_rows, T, k0, wave, w, out);
}

}  // extern "C"
