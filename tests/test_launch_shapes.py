"""Which launches a call makes: their number, order and sizes, on the CPU.  The library's launches are caught by a hipLaunchKernel of
this test's own, loaded before the runtime's, so the real argument checks, rules and dispatch run with pointers that nobody follows.
The rules are those for 256 CUs (what the library takes a machine for that does not tell)."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CATCH = r"""
#include <stdio.h>
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim;
static dim grid, block;
int __hipPushCallConfiguration(dim g, dim b, size_t lds, void* stream) { grid = g; block = b; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* lds, void** stream) { *g = grid; *b = block; *lds = 0; *stream = NULL; return 0; }
int hipLaunchKernel(const void* f, dim g, dim b, void** args, size_t lds, void* stream) {
  printf("launch %u %u %u %u\n", g.x, g.y, g.z, b.x * b.y * b.z);
  fflush(stdout);
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 100; }
"""

CALLS = r"""
import ctypes, json, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2408_10188_amd import binding as B
for line in sys.stdin:
    c = json.loads(line)
    P = 1 << 20
    d, hq, hkv, rows = c["d"], c["hq"], c["hkv"], c["n_q"]
    shape = B.make_shape(hq, hkv, d, B.MMSP_F32 if c["f32"] else B.MMSP_BF16, d ** -0.5, (hq * d, d), (hkv * d, d), rows)
    blk = B.make_block(0, rows, 0, c["n_k"], c["mask"], c["pos"], 0, P if c["docs"] else None, c["docs"])
    ws = c["ws"] if c["ws"] >= 0 else B.mmsp_workspace_bytes(shape, rows, c["n_k"], True)
    if c["what"] == "fwd":
        B.mmsp_attn_step_fwd(shape, blk, P, P, P, P, P, c["accumulate"], P if ws else None, ws)
    else:
        dq, dk = (P if x in c["what"] else None for x in ("dq", "dk"))
        B.mmsp_attn_step_bwd(shape, blk, P, P, P, None, P, P, P, False, dq, dk, dk, False, P, ws)
    print("end", flush=True)
"""


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("catch")
    src, so, calls = tmp / "catch.c", tmp / "catch.so", tmp / "calls.py"
    src.write_text(CATCH)
    calls.write_text(CALLS)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    p = subprocess.Popen([sys.executable, str(calls), str(so), ROOT], stdin=subprocess.PIPE, stdout=subprocess.PIPE, text=True)
    yield p
    p.stdin.close()
    assert p.wait(timeout=60) == 0


def launches(library, what, hq, hkv, n_q, n_k, mask=0, pos=0, docs=0, d=128, f32=False, ws=-1, accumulate=False):
    """[(workgroups along x, y, z, threads of one)] of a call; ws: bytes of workspace, -1: what the backward asks for."""
    library.stdin.write(json.dumps(dict(what=what, hq=hq, hkv=hkv, n_q=n_q, n_k=n_k, mask=mask, pos=pos, docs=docs, d=d, f32=f32, ws=ws,
                                        accumulate=accumulate)) + "\n")
    library.stdin.flush()
    got = []
    while True:
        line = library.stdout.readline().split()
        assert line, "the call failed"
        if line[0] == "end":
            return got
        got.append(tuple(int(x) for x in line[1:]))


@pytest.mark.parametrize("what", ["fwd", "dq", "dk", "dq dk"])
@pytest.mark.parametrize("hq,hkv,n_q,n_k", [(32, 32, 1 << 22, 16), (32, 32, 16, 1 << 22), (2, 1, 1 << 26, 16)])
def test_a_grid_dimension_holds_fewer_than_2_32_threads(library, what, hq, hkv, n_q, n_k):
    """2^27 (row, head)s of fp32 at d = 64 are 34 GB a tensor, and 2^23 workgroups of 512 threads: one dimension of a grid takes one fewer."""
    for f32, d in ((True, 64), (False, 128)):
        got = launches(library, what, hq, hkv, n_q, n_k, d=d, f32=f32)
        assert got
        for x, y, z, threads in got:
            assert x * threads < 1 << 32 and y < 1 << 16 and z == 1


@pytest.mark.parametrize("what", ["fwd", "dq"])
def test_rows_of_a_small_block_are_spread_over_the_chip(library, what):
    """Tiles of 32 (row, head) pairs where they fit the CUs, then of 64 and 128; four wavefronts in each."""
    for hq, hkv, n_q, n_k, tiles in [(28, 4, 50, 50, 11), (28, 4, 300, 64, 66 // 2), (28, 4, 600, 64, 33), (8, 8, 500, 64, 16), (4, 2, 1, 64, 1)]:
        (x, y, z, threads), = launches(library, what, hq, hkv, n_q, n_k, 0)
        per_head = 8 // hkv                                # XCDs of a KV head share its tiles evenly
        assert (x, threads) == (8 * -(-tiles // per_head), 256), (hq, hkv, n_q)
