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
    blk = B.make_block(0, rows, 0, c["n_k"], c["mask"], c["pos"], c["k_pos"], P if c["docs"] else None, c["docs"])
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


def launches(library, what, hq, hkv, n_q, n_k, mask=0, pos=0, docs=0, d=128, f32=False, ws=-1, accumulate=False, k_pos=0):
    """[(workgroups along x, y, z, threads of one)] of a call; ws: bytes of workspace, -1: what the backward asks for."""
    library.stdin.write(json.dumps(dict(what=what, hq=hq, hkv=hkv, n_q=n_q, n_k=n_k, mask=mask, pos=pos, k_pos=k_pos, docs=docs, d=d, f32=f32,
                                        ws=ws, accumulate=accumulate)) + "\n")
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
    """Tiles of 8 (row, head) pairs where they fit the CUs, then of 16 to 128; four wavefronts in each."""
    for hq, hkv, n_q, n_k, tiles in [(28, 4, 50, 50, 44), (28, 4, 300, 64, 33), (28, 4, 600, 64, 33), (8, 8, 500, 64, 32), (4, 2, 1, 64, 1)]:
        (x, y, z, threads), = launches(library, what, hq, hkv, n_q, n_k, 0)
        per_head = 8 // hkv                                # XCDs of a KV head share its tiles evenly
        assert (x, threads) == (8 * -(-tiles // per_head), 256), (hq, hkv, n_q)


@pytest.mark.parametrize("what", ["fwd", "dq"])
@pytest.mark.parametrize("hq,hkv,n_q,tiles,docs", [(7, 1, 4961, 136, 0), (8, 8, 4283, 17, 0), (7, 1, 5651, 155, 2)])
def test_keys_under_a_causal_mask_are_cut_though_not_in_whole_rounds(library, what, hq, hkv, n_q, tiles, docs):
    """Half of the pairs are hidden, so a launch of one and a half rounds lasts little longer than one of half a round: 73 us instead of 104 (4961 rows of 7/1 heads, forward)."""
    assert launches(library, what, hq, hkv, n_q, n_q, 1, docs=docs)[0][0] > 256 > 8 * -(-tiles // (8 // hkv))


def shares(library, hkv, n_k, got):
    """Shares of a key tile that the launches of a dK/dV call dealt out."""
    tiles, per_head = -(-n_k // 128), 8 // hkv
    blocks = [x for x, y, z, threads in got if y == 1][-1]                      # the reduction is a grid of two rows
    counts = [n for n in range(1, 33) if 8 * -(-tiles * n // per_head) == blocks]
    assert (len(got) == 3) == (counts[-1] > 1)                                  # row statistics, the kernel, the reduction
    return counts


@pytest.mark.parametrize("hq,hkv,n_q,behind,want", [
    (28, 4, 300, 3000, 2), (28, 4, 500, 3000, 2), (28, 4, 1000, 3000, 2),       # whole rounds of tiles that see all rows: 50, 65, 111 us; three shares 67, 87, 142
    (7, 1, 1000, 3000, 8), (14, 2, 500, 10000, 1), (28, 4, 1000, 0, 8),         # 45 (eleven: 60), 90 (two: 114), 40 us (six: 44)
    (7, 1, 2500, 0, 16),                                                        # a triangle: more shares than eight, 49 us (eight: 65)
])
def test_shares_go_by_what_the_key_tiles_see(library, hq, hkv, n_q, behind, want):
    assert want in shares(library, hkv, n_q + behind, launches(library, "dk", hq, hkv, n_q, n_q + behind, 1, behind))


def test_shares_of_several_documents_suit_a_long_one_too(library):
    """26 documents of 4000 keys: many of 150, or one of 3500 with clips.  One share per tile, which suits the first, takes 221 us of the second, eight 76 us."""
    assert 8 in shares(library, 2, 4000, launches(library, "dk", 4, 2, 4000, 4000, 1, 0, docs=26))
    # two KV heads see whole documents of known length
    one = shares(library, 2, 4000, launches(library, "dk", 4, 2, 4000, 4000, 1, 0, docs=1))
    assert one == shares(library, 2, 4000, launches(library, "dk", 4, 2, 4000, 4000, 1, 0))


@pytest.mark.parametrize("case,want", [
    # blocks that tests/test_gpu_row_lists.py runs on the GPU, and the routes that they mean to take
    (dict(what="dk", hq=7, hkv=1, n_q=1300, n_k=130), 32), (dict(what="dk", hq=7, hkv=1, n_q=1100, n_k=1100, mask=1), 18),
    (dict(what="dk", hq=5, hkv=5, n_q=70, n_k=900, mask=1, pos=830), 1),
])
def test_shares_of_the_gpu_tests(library, case, want):
    got = launches(library, **case)
    if case["hkv"] == 5:
        assert [g[0] for g in got if g[1] == 1] == [8 * 5]                       # key tiles x KV heads, one share each
    else:
        assert want in shares(library, case["hkv"], case["n_k"], got)


@pytest.mark.parametrize("hq,hkv,n_q,n_k,want", [
    (2, 1, 37, 41, [3 + 3 + 6]), (8, 2, 399, 401, [52 + 52 + 200]),              # dK and dV apart from each other
    (8, 8, 120, 250, [128 + 64]), (8, 8, 257, 259, [17 * 8, 17 * 8]),            # together in one launch; two launches
])
def test_launches_of_the_fp32_gradients(library, hq, hkv, n_q, n_k, want):
    assert [x * y for x, y, z, t in launches(library, "dq dk", hq, hkv, n_q, n_k, d=64, f32=True)] == want


def test_workgroups_of_eight_wavefronts_in_the_gpu_tests(library):
    """tests/test_gpu_row_lists.py runs 1190 rows of 28/4 heads for the wide workgroups: 33 tiles of 256 pairs per KV head, which two XCDs share."""
    for n_k in (1, 64, 130, 257):
        assert launches(library, "fwd", 28, 4, 1190, n_k) == launches(library, "dq", 28, 4, 1190, n_k) == [(8 * 17, 1, 1, 512)]
