// The LDS maps of csrc/lds_tiles.h for the host, by row size: what tests/test_lds_direct_maps.py checks.
#include "lds_tiles.h"

template <typename F>
static int by_row(int row, F f)
{
    switch (row) {
    case 64: return f.template of<64>();
    case 128: return f.template of<128>();
    case 256: return f.template of<256>();
    case 512: return f.template of<512>();
    }
    return -1;
}

#define MAP(name, expr)                                                                                        \
    struct name##_of {                                                                                         \
        int a, b;                                                                                              \
        template <int ROW>                                                                                     \
        int of() const { return expr; }                                                                        \
    };                                                                                                         \
    extern "C" int name(int row, int a, int b) { return by_row(row, name##_of{a, b}); }

MAP(map_swizzle_k, dream::swizzle_k<ROW>(a))
MAP(map_swizzle_v, dream::swizzle_v<ROW>(a))
MAP(map_piece_k, dream::piece_k<ROW>(a))
MAP(map_piece_v, dream::piece_v<ROW>(a))
MAP(map_fragment_k, dream::fragment_k<ROW>(a, b))
MAP(map_fragment_v, dream::fragment_v<ROW>(a, b))
extern "C" int map_at_key_step(int fragment, int ks) { return dream::at_key_step(fragment, ks); }
extern "C" int map_at_column_tile(int fragment, int dt) { return dream::at_column_tile(fragment, dt); }
extern "C" int map_turned_step(int i, int n_steps, int turned) { return dream::turned_step(i, n_steps, turned); }
extern "C" int map_turn() { return dream::TURN; }
