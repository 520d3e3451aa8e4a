"""Where the asynchronous tile copies land: their LDS target is a register that the source computes, so it is read off the generated code
of a kernel with a second array in front of the tiles."""
import os
import re
import subprocess

import pytest

from paper_2408_10188_amd import build

KERNEL = """
#include "mfma_tiles.h"
using namespace mmsp;
__global__ __launch_bounds__(64) void copies(const char* from, int* out) {
  __shared__ __attribute__((aligned(4096))) int other[2048];          // the stricter alignment goes first: addresses 0 .. 8191
  __shared__ __attribute__((aligned(1024))) char tiles[2 * kTileGBytes];
  other[threadIdx.x] = out[threadIdx.x];
  TileCopier<16> c;
  c.init(tiles, 128, 64, 0, 0, threadIdx.x);
  const auto t = c.tile(from, 0);
  c.copy(t, 3, kTileGBytes);
  c.copy_to(t, 5, kTileGBytes);
  dma16(from, threadIdx.x * 16, tiles, 4096);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  out[threadIdx.x] = other[threadIdx.x ^ 1] + reinterpret_cast<const int*>(tiles)[threadIdx.x];
}
"""


def targets(asm):
    """Values that M0 is set to, from the constants in scalar registers."""
    value, out = {}, []
    for line in asm:
        m = re.match(r"\s+(s_\w+)\s+(\w+), (\w+)(?:, (\w+))?", line)
        if not m:
            continue
        op, to, *args = m.groups()
        args = [value.get(x) if x[0] == "s" else int(x, 0) for x in args if x is not None]
        result = None if None in args else args[0] if op.startswith("s_mov") else sum(args) if op.startswith("s_add_i32") else None
        value[to] = result
        if to == "m0":
            out.append(result)
    return out


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
def test_copies_go_to_their_array(tmp_path):
    src, out = tmp_path / "copies.hip", tmp_path / "copies.s"
    src.write_text(KERNEL)
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "-I" + build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    group, tile = 1040, 16 * 1040                         # bytes of four rows, of a slot
    assert targets(out.read_text().splitlines()) == [8192 + tile + 3 * group, 8192 + tile + 5 * group, 8192 + 4096]
