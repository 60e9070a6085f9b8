"""How a package of escape-time rows is cut into the waves' blocks of 64 pixels
(common.hpp, shared by the engine and its kernels): the blocks cover the package,
and a wave's work is pixels, not padding, however few rows a package has."""
import os
import subprocess

import pytest

from test_kernel_isa import CSRC

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "common.hpp"
int main(int, char** a) {
  const uint32_t w = (uint32_t)strtoull(a[1], 0, 0);
  for (uint64_t rows = 1; rows <= 40; ++rows) {
    const uint32_t bits = ce::escape_block_bits(rows);
    printf("%llu %u %llu %llu\n", (unsigned long long)rows, bits, (unsigned long long)ce::escape_blocks_across(w, bits),
           (unsigned long long)ce::escape_blocks_down(rows, bits));
  }
}
"""


@pytest.mark.parametrize("w", [1, 15, 16, 17, 63, 64, 65, 1000, 8192, 0xFFFFFFFF])
def test_blocks_cover_the_package_without_padding_rows(tmp_path, w):
    src = tmp_path / "blocks.cpp"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "blocks"), str(src)], check=True)
    out = subprocess.run([str(tmp_path / "blocks"), str(w)], check=True, capture_output=True, text=True).stdout
    rows_seen = 0
    for line in out.splitlines():
        rows, bits, across, down = (int(x) for x in line.split())
        cols, high = 1 << bits, 64 >> bits
        assert cols * high == 64
        assert (across - 1) * cols < w <= across * cols
        assert (down - 1) * high < rows <= down * high
        assert down * high * 3 <= rows * 5, (rows, high)  # of 3 and 5 rows a third and three fifths are padding
        if rows <= 2:
            assert down * high == rows
        rows_seen += 1
    assert rows_seen == 40


HOST_SRC = r"""
#include <cstdio>
#include "common.hpp"
int main() {
  const uint32_t sides[][2] = {{1, 1}, {31, 400}, {32, 400}, {63, 400}, {64, 64}, {200, 200}, {512, 512}, {1024, 1024},
                               {2048, 2048}, {4099, 3001}, {100, 100000}, {8192, 8192}};
  for (auto& s : sides) {
    const uint32_t bits = ce::blur_tile_row_bits(s[0], s[1], true);
    printf("%u %u %u %u %llu\n", s[0], s[1], ce::escape_block_bits(400, ce::escape_least_bits(s[0], true)), 1u << bits,
           (unsigned long long)(ce::ceil_div(s[1], 1ull << bits) * ce::ceil_div(s[0], ce::kBlurTileCols)));
  }
}
"""


def test_tiles_of_host_memory_suit_the_link(tmp_path):
    """Buffers in pinned host memory: escape-time blocks are rows of 64 pixels as
    far as the image is that wide, and blur tiles short only until there are
    32 of them (each reads four halo rows over the link)."""
    src = tmp_path / "host.cpp"
    src.write_text(HOST_SRC)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "host"), str(src)], check=True)
    out = subprocess.run([str(tmp_path / "host")], check=True, capture_output=True, text=True).stdout
    lines = [[int(x) for x in line.split()] for line in out.splitlines()]
    assert len(lines) == 12
    for w, h, bits, rows, tiles in lines:
        assert bits == (6 if w >= 64 else 5 if w >= 32 else 4)
        assert rows in (2, 4, 8, 16, 32)
        assert rows == 32 or tiles < 64
        assert rows == 2 or tiles >= 32


DEEP_SRC = r"""
#include <cstdio>
#include "common.hpp"
int main() {
  const uint32_t calls[][3] = {{64, 64, 1}, {64, 64, 1024}, {64, 64, 1025}, {40, 64, 1024}, {20, 64, 1}, {4096, 2047, 1025},
                               {4096, 2048, 1025}, {4096, 2048, 4096}, {4096, 2048, 4097}, {65536, 65536, 4096}};
  for (auto& c : calls) printf("%u %u ", ce::escape_least_bits(c[0], c[1], c[2], true), ce::escape_least_bits(c[0], c[1], c[2], false));
}
"""


def test_deep_caps_keep_square_blocks(tmp_path):
    """A wave of 64 pixels in a row lasts as long as its longest orbit: into host
    memory rows are taken up to max_iter 1024 only, 4096 from 2^23 pixels on."""
    src = tmp_path / "deep.cpp"
    src.write_text(DEEP_SRC)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "deep"), str(src)], check=True)
    out = subprocess.run([str(tmp_path / "deep")], check=True, capture_output=True, text=True).stdout.split()
    assert [int(x) for x in out[::2]] == [6, 6, 4, 5, 4, 4, 6, 6, 4, 6]
    assert [int(x) for x in out[1::2]] == [4] * 10
