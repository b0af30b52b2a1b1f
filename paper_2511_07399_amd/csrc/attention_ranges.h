// The key tiles of one part of an attention launch.  Without dependencies: the kernels and the host use it.
#pragma once

namespace sdv2 {

struct KeyTiles {
    int first, full, end;      // tiles [first, full) hold only valid keys; tile `full`, where full < end, has slots past them
};

// Part `part` of `parts` (at most 16: no overflow of 32 bits below 2^33 keys) of kv_len > 0 keys in tiles of `tile`.  Parts beyond
// the number of tiles are empty, the first ones among them: then first = full = end.
constexpr KeyTiles key_tiles(int kv_len, int tile, int part, int parts) {
    const int n = (int)((unsigned)(kv_len + tile - 1) / (unsigned)tile);
    KeyTiles t{0, n, n};
    if (parts > 1) {
        t.first = (int)((unsigned)(part * n) / (unsigned)parts);
        t.end = (int)((unsigned)((part + 1) * n) / (unsigned)parts);
    }
    const int short_end = (unsigned)kv_len % (unsigned)tile != 0 ? n : -1;      // where a part ends whose last tile is short
    t.full = t.end == short_end ? t.end - 1 : t.end;                            // such a part has a tile
    return t;
}

}  // namespace sdv2
