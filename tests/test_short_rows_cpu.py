"""The short-row kernels' LDS: what a launch asks for holds every entry that a lane reads, its own or not.  The sizes come
from the header that the launches use, built for the host; the reads are walked through here lane by lane."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_18513_amd", "csrc")


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    folder = tmp_path_factory.mktemp("short_rows")
    src, so = folder / "layout.cpp", folder / "layout.so"
    src.write_text('#include "short_rows.hpp"\n'
                   'extern "C" long lds(int cols, int k, int G, int esz, int block) { return (long)slimfit::short_lds_bytes(cols, k, G, esz, block); }\n'
                   'extern "C" long rows(int cols, int G, int esz) { return (long)slimfit::short_rows_bytes(cols, G, esz); }\n'
                   'extern "C" int held_block() { return slimfit::kShortHeldBlock; }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.lds.restype = lib.rows.restype = ctypes.c_long
    return lib


def _furthest_byte(cols, G, esz, block):
    """One past the last byte that a lane of the wave reads of the staged rows."""
    part = -(-cols // G)
    last_row = (64 // G - 1) * cols
    return max((last_row + q * part + -(-part // block) * block) * esz for q in range(G))


@pytest.mark.parametrize("G,esz,held", [(8, 4, True), (4, 4, True), (4, 2, True), (2, 2, True), (4, 4, False), (2, 2, False)])
def test_every_read_is_inside_the_launch(layout, G, esz, held):
    block = layout.held_block() if held else 1
    for cols in range(1, 257):
        rows_end = 64 // G * cols * esz
        assert layout.rows(cols, G, esz) >= rows_end and layout.rows(cols, G, esz) % 16 == 0
        for k in range(1, min(cols, 16) + 1):
            lds = layout.lds(cols, k, G, esz, block)
            assert lds >= _furthest_byte(cols, G, esz, block), (cols, k)
            assert lds >= layout.rows(cols, G, esz) + 64 // G * k * 4, (cols, k)
            assert lds <= 160 * 1024


def test_the_rows_and_the_slots_alone_were_too_little(layout):
    """Eight lanes a row, one entry kept: the eight slots behind the rows are less than the ten entries read there."""
    for cols in (97, 129, 161, 193, 225):
        assert layout.rows(cols, 8, 4) + 8 * 4 < _furthest_byte(cols, 8, 4, 4) <= layout.lds(cols, 1, 8, 4, 4)
