"""Host-side check of the addresses that the dense pass over X asks for (no GPU needed).

`csrc/dense_reads.h` states the buffer and the lane offset of every tile load as plain arithmetic; the kernel uses the
same functions.  A small program compiled from that header walks all tiles (those beyond the matrix included), strips
and lanes of small and odd sizes, and applies the documented rule of a raw buffer load: a dword is read if its offset
from voffset lies below the buffer's range, whatever soffset is; its address is base + soffset + voffset.  No dword may
be read outside the tensor, and what belongs to the matrix has to be read, at its own place.  The same walk with the
tile column in soffset (a mistake that the kernel once had) reads behind the tensor: that is what makes the check worth
something."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "dense_reads.h"
#include <cstdio>
#include <cstdlib>
using namespace nnr;

// dwords read outside the tensor, and (returned in wrong) dwords of the matrix that are not read or read elsewhere
static long walk(int64_t n, int m, int waves, bool in_soffset, long& wrong) {
  const int64_t total = (int64_t)m * n * n, panels = (n + 16 * waves - 1) / (16 * waves);
  long outside = 0;
  for (int t = 0; t < m; ++t)
    for (int64_t panel = 0; panel < panels; ++panel)
      for (int64_t i0 = 0; i0 < n; i0 += 16) {
        const int64_t jp0 = panel * 16 * waves;
        const TileBuffer b = tile_buffer(n, total, t, i0, jp0);
        for (int jt = 0; jt < waves; ++jt)
          for (int lane = 0; lane < 64; ++lane) {
            const int l16 = lane & 15, row = lane >> 4;
            const uint32_t lo = tile_lane_offset((uint32_t)n, l16, row);
            const uint32_t voffset = in_soffset ? lo : tile_voffset(lo, jt), soffset = in_soffset ? 64u * jt : 0u;
            for (int r = 0; r < 4; ++r) {
              const bool read = (uint64_t)voffset + 4 * r < b.bytes;
              const int64_t at = 4 * b.first + soffset + voffset + 4 * r;
              if (read && (at < 0 || at >= 4 * total)) ++outside;
              const int64_t i = i0 + l16, j = jp0 + 16 * jt + 4 * row + r;
              if (i < n && j < n && !(read && at == 4 * ((t * n + i) * n + j))) ++wrong;
            }
          }
      }
  return outside;
}

int main(int argc, char** argv) {
  long wrong = 0;
  const long outside = walk(atoll(argv[1]), atoi(argv[2]), atoi(argv[3]), argv[4][0] == '1', wrong);
  printf("%ld %ld\n", outside, wrong);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    folder = tmp_path_factory.mktemp("dense_reads")
    src, exe = folder / "walk.cpp", folder / "walk"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2202_09512_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def run(n, m, waves, in_soffset):
        out = subprocess.run([str(exe), str(n), str(m), str(waves), "1" if in_soffset else "0"], check=True,
                             capture_output=True, text=True).stdout
        return [int(v) for v in out.split()]
    return run


@pytest.mark.parametrize("waves", [4, 8])
def test_no_tile_load_leaves_the_tensor(walk, waves):
    for n in [1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 112, 127, 128, 129, 130, 255, 257, 333]:
        for m in (1, 3):
            assert walk(n, m, waves, False) == [0, 0], (n, m)


def test_walk_catches_a_tile_column_that_is_not_compared(walk):
    for n, m in [(17, 1), (32, 1), (112, 2)]:
        outside, _ = walk(n, m, 8, True)
        assert outside > 0, (n, m)
    assert walk(256, 1, 8, True) == [0, 0]         # whole panels: nothing beyond the matrix is asked for
