// Where the 16-byte pieces of key and value tiles lie in LDS (attend_rows in attn.hip): plain integer arithmetic, also compiled for the host by the
// test of these maps.  ROW: bytes of a tile's row.  A load instruction moves 64 pieces, lane i's to 16 * i behind the instruction's 1024 bytes, so a row's pieces are
// swapped by choosing which one a lane reads.
#pragma once

namespace dream {

// The byte of its row that lane's piece of load instruction 0 comes from; of instruction j it is that ^ swizzle_k(j), swizzle_v(j).
// K: piece i of row r sits at i ^ (r mod 16) (rows of 128 bytes, two to a bank line: i ^ (r/2 mod 8)).
template <int ROW>
constexpr int swizzle_k(int j) { return ROW == 128 ? ((j * 4) & 7) * 16 : ((j * (1024 / ROW)) & 15) * 16; }
template <int ROW>
constexpr int piece_k(int lane)
{
    const int row = lane / (ROW / 16);
    return ((lane % (ROW / 16)) ^ (ROW == 128 ? row >> 1 : row)) * 16;
}
// V: pair i of the pieces of row r sits at i ^ pair_of_v(r)
template <int ROW>
constexpr int swizzle_v(int j) { return ROW <= 128 ? 0 : ((j * (1024 / ROW)) & 7) * 32; }
template <int ROW>
constexpr int pair_of_v(int r) { return ROW == 64 ? (r >> 2) & 1 : ROW == 128 ? (r >> 1) & 3 : r & 7; }
template <int ROW>
constexpr int piece_v(int lane) { return ((lane % (ROW / 16)) ^ (2 * pair_of_v<ROW>(lane / (ROW / 16)))) * 16; }

// Where lane (c, g) reads its K fragment (row c, 16 bytes) of key step 0 of a 16-row half, and the one of step ks from there
template <int ROW>
constexpr int fragment_k(int c, int g) { return c * ROW + ((g ^ (ROW == 128 ? c >> 1 : c)) * 16); }
constexpr int at_key_step(int fragment, int ks) { return (fragment ^ ((ks & 3) * 64)) + (ks >> 2) * 256; }
// Where it reads its share of the transposing read of V (row 4 g + c/4, 8 bytes) of column tile 0, and of column tile dt
template <int ROW>
constexpr int fragment_v(int c, int g)
{
    const int row = g * 4 + (c >> 2);
    return row * ROW + pair_of_v<ROW>(row) * 32 + (c & 3) * 8;
}
constexpr int at_column_tile(int fragment, int dt) { return (fragment ^ ((dt & 7) * 32)) + (dt >> 3) * 256; }


// The step that a workgroup which is `turned` (0 .. TURN - 1) takes as its i-th of n_steps: of every TURN steps behind the first, another one first and then round.
constexpr int TURN = 8;
constexpr int turned_step(int i, int n_steps, int turned)
{
    if (i <= 0)
        return i;
    const int at = (unsigned)(i - 1) % TURN, first = i - at, n = n_steps - first < TURN ? n_steps - first : TURN, k = at + (unsigned)(turned * n) / TURN;
    return first + (k < n ? k : k - n);
}

}  // namespace dream
