"""Host model of the LDS layout of the attention kernels whose tiles go from memory straight to LDS (attend_rows in csrc/attn.hip; the
areas in test_lds_index_maps.py are those of tiles staged in registers).  The address maps are the kernel's own (csrc/lds_tiles.h, built for the host); this
file says what they have to do: where every lane of a load instruction puts its 16 bytes, where the fragment reads look for them, and which banks the lanes of a read
touch together."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module", autouse=True)
def maps(tmp_path_factory):
    """tests/c/lds_tiles_check.cpp, which instantiates the header's templates for every row size."""
    out = str(tmp_path_factory.mktemp("maps") / "lds_tiles_check.so")
    csrc = os.path.join(os.path.dirname(HERE), "paper_2505_19201_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-I" + csrc, os.path.join(HERE, "c", "lds_tiles_check.cpp"), "-o", out], check=True)
    global LIB
    LIB = ctypes.CDLL(out)


def swizzle_k(row_bytes, j):
    return LIB.map_swizzle_k(row_bytes, j, 0)


def swizzle_v(row_bytes, j):
    return LIB.map_swizzle_v(row_bytes, j, 0)


def loaded(row_bytes, keys, kind):
    """LDS byte -> (row, byte of the row) after the loads of one tile."""
    lanes = row_bytes // 16
    at = {}
    for j in range(keys * row_bytes // 1024):
        for lane in range(64):
            row = lane // lanes
            if kind == "k":
                chunk = LIB.map_piece_k(row_bytes, lane, 0) ^ swizzle_k(row_bytes, j)
            else:
                chunk = LIB.map_piece_v(row_bytes, lane, 0) ^ swizzle_v(row_bytes, j)
            assert 0 <= chunk < row_bytes
            for i in range(0, 16, 2):
                at[j * 1024 + lane * 16 + i] = (j * (64 // lanes) + row, chunk + i)
    assert sorted(at) == list(range(0, keys * row_bytes, 2))
    assert len(set(at.values())) == len(at)          # every element of the tile once
    return at


@pytest.mark.parametrize("row_bytes,keys,kind", [(256, 32, "k"), (512, 16, "k"), (256, 32, "v"), (256, 16, "v")])
def test_two_loaders_put_the_tile_where_one_does(row_bytes, keys, kind):
    """The second loader's instructions, its half of the rows further, with the half's own bit of the swizzle in the lane's chunk."""
    lanes, at = row_bytes // 16, {}
    n = keys * row_bytes // 1024 // 2
    swizzle = swizzle_k if kind == "k" else swizzle_v
    for half in range(2):
        for j in range(n):
            for lane in range(64):
                row = lane // lanes
                own = (LIB.map_piece_k if kind == "k" else LIB.map_piece_v)(row_bytes, lane, 0) ^ half * swizzle(row_bytes, n)
                for i in range(0, 16, 2):
                    at[half * n * 1024 + j * 1024 + lane * 16 + i] = (half * n * (64 // lanes) + j * (64 // lanes) + row, (own ^ swizzle(row_bytes, j)) + i)
    assert at == loaded(row_bytes, keys, kind)


def bank_groups(addresses, width):
    """Lanes served together: 256 bytes of the 64 banks at a time."""
    per = 256 // width
    for first in range(0, 64, per):
        yield [(a // 4 + w) % 64 for a in addresses[first:first + per] for w in range(width // 4)]


@pytest.mark.parametrize("D,keys", [(64, 32), (128, 16), (128, 32), (256, 16), (256, 32)])
def test_key_fragments(D, keys):
    row_bytes = 2 * D
    at = loaded(row_bytes, keys, "k")
    for h in range(keys // 16):
        for ks in range(D // 32):
            addresses = []
            for lane in range(64):
                c, g = lane & 15, lane >> 4
                a = h * 16 * row_bytes + LIB.map_at_key_step(LIB.map_fragment_k(row_bytes, c, g), ks)
                addresses.append(a)
                for e in range(8):               # lane (c, g): key c of the half, dimensions 32 ks + 8 g ..
                    assert at[a + 2 * e] == (h * 16 + c, (ks * 32 + g * 8 + e) * 2)
            for banks in bank_groups(addresses, 16):
                assert len(set(banks)) == len(banks)


@pytest.mark.parametrize("DV,keys", [(32, 16), (32, 32), (64, 16), (64, 32), (128, 16), (128, 32), (256, 16)])
def test_value_fragments(DV, keys):
    row_bytes = 2 * DV
    at = loaded(row_bytes, keys, "v")
    for h in range(keys // 16):
        for dt in range(DV // 16):
            addresses = []
            for lane in range(64):
                c, g = lane & 15, lane >> 4
                row = g * 4 + (c >> 2)
                a = h * 16 * row_bytes + LIB.map_at_column_tile(LIB.map_fragment_v(row_bytes, c, g), dt)
                addresses.append(a)
                for e in range(4):               # the transposing read takes 4 columns of row g*4 + c/4 from lane (c, g)
                    assert at[a + 2 * e] == (h * 16 + row, (dt * 16 + (c & 3) * 4 + e) * 2)
            for banks in bank_groups(addresses, 8):
                assert len(set(banks)) == len(banks)


def test_turned_steps_are_an_order_of_all_steps():
    """Every step once, the first one first, whatever the number of steps and the workgroup; the workgroups of a head start the steps behind it apart."""
    turn = LIB.map_turn()
    for n in range(1, 70):
        for workgroups in (3, 4, 5, 8, 10, 12, 32):
            starts = set()
            for unit in range(workgroups):
                turned = unit * ((turn << 16) // workgroups) >> 16
                assert 0 <= turned < turn
                order = [LIB.map_turned_step(i, n, turned) for i in range(n)]
                assert order[0] == 0 and sorted(order) == list(range(n)), (n, turned, order)
                starts.add(order[1] if n > 1 else 0)
            assert len(starts) >= (min(workgroups, turn) if n > turn else 2 if n > 2 else 1), (n, workgroups)
