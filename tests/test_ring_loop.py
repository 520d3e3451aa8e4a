"""The host loop of ring.py by itself: which rows its calls leave how, and what it holds while they run.  The calls of the library are
replaced by recorders, so no GPU is needed; layouts and plans are the library's own."""
import types
import weakref

import numpy as np
import pytest
import torch

from paper_2408_10188_amd import binding as B
from paper_2408_10188_amd import ring


class Rows:
    """Stands for the step calls: per row of the output 'old', 'empty' (nothing visible) or 'result'."""

    def __init__(self, n_rows):
        self.state = ["old"] * n_rows

    def binding(self):
        fake = types.SimpleNamespace(**{n: getattr(B, n) for n in dir(B) if not n.startswith("__")})
        fake.mmsp_attn_step_fwd, fake.mmsp_attn_merge = self.step_fwd, lambda *a, **k: None
        return fake

    def step_fwd(self, shape, blk, q, k, v, o, lse, accumulate, ws=None, ws_bytes=0, stream=0):
        for i in range(blk.q_row0, min(blk.q_row0 + blk.n_q, len(self.state))):
            nothing = blk.mask == B.MMSP_MASK_NONE or blk.n_k == 0
            if nothing and not accumulate:
                self.state[i] = "empty"
            elif not nothing:
                assert not accumulate or self.state[i] != "old", "row %d is merged into what no call has written" % i
                self.state[i] = "result"


@pytest.mark.parametrize("extra", [0, 1, 32, 200])
@pytest.mark.parametrize("N,rank", [(1, 0), (2, 1), (3, 0)])
def test_rows_behind_a_packed_ranks_own_are_empty(monkeypatch, N, rank, extra):
    """A query buffer longer than the rank's 2C rows: these have a result, the rows behind them an empty one."""
    C = 64
    rows = Rows(2 * C + extra)
    monkeypatch.setattr(ring, "B", rows.binding())
    cu_host = np.array([0, 40, 2 * N * C], dtype=np.int32)
    cu = torch.from_numpy(cu_host)
    q = torch.zeros(2 * C + extra, 2, 128, dtype=torch.bfloat16)
    k = torch.zeros(N, 2 * C, 1, 128, dtype=torch.bfloat16)
    shape = ring.shape_for(q, k, B.MMSP_BF16, 2 * C + extra)
    o, lse = torch.zeros(2 * C + extra, 2, 128), torch.zeros(2, 2 * C + extra)
    for host in (None, cu_host):
        ring.rank_forward_packed(shape, 2 * N * C, N, rank, q, k, k, cu, 2, o, lse, cu_host=host)
        assert rows.state == ["result"] * (2 * C) + ["empty"] * extra
        rows.state = ["old"] * len(rows.state)


class Made:
    """A sequence of blocks that are made when asked for, as a program does that receives them one by one."""

    def __init__(self, only, *size):
        self.only, self.size, self.alive, self.asked = only, size, {}, []

    def __getitem__(self, r):
        if r not in self.only:
            raise KeyError(r)
        t = torch.zeros(self.size, dtype=torch.bfloat16)
        self.alive[t.data_ptr()] = weakref.ref(t)
        self.asked.append(r)
        return t

    def holds(self, address):
        return address in self.alive and self.alive[address]() is not None


class Stream:
    cuda_stream = 0

    def __init__(self, waiting=lambda: None):
        self.waiting = waiting

    def wait_stream(self, other):
        self.waiting()


def _pass(monkeypatch, blocks, N, rank, C, call, side=None, packed=None):
    """One forward and one backward pass with every call replaced by `call(k, v, dk)`."""
    fake = types.SimpleNamespace(**{n: getattr(B, n) for n in dir(B) if not n.startswith("__")})
    fake.mmsp_attn_step_fwd = lambda shape, blk, q, k, v, *a, **kw: call(k, v)
    fake.mmsp_attn_step_bwd = lambda shape, blk, q, k, v, *a, **kw: call(k, v)
    fake.mmsp_attn_merge = fake.mmsp_attn_delta = lambda *a, **kw: None
    monkeypatch.setattr(ring, "B", fake)
    q, o, lse = torch.zeros(2 * C, 2, 128, dtype=torch.bfloat16), torch.zeros(2 * C, 2, 128), torch.zeros(2, 2 * C)
    shape = ring.shape_for(q, torch.zeros(2 * C, 1, 128), B.MMSP_BF16, 2 * C)
    dk = torch.zeros(N, 2 * C, 1, 128)
    T = 2 * N * C
    if packed is not None:
        docs = torch.from_numpy(packed), len(packed) - 1
        ring.rank_forward_packed(shape, T, N, rank, q, *blocks, *docs, o, lse, cu_host=packed)
        ring.rank_backward_packed(shape, T, N, rank, q, *blocks, *docs, q, q, lse, lse, o, dk, dk, cu_host=packed)
    else:
        ring.rank_forward(shape, T, N, rank, q, *blocks, o, lse, side=side)
        ring.rank_backward(shape, T, N, rank, q, *blocks, q, q, lse, lse, o, dk, dk, side=side)


@pytest.mark.parametrize("packed", [False, True])
def test_blocks_made_on_demand_live_until_their_launch(monkeypatch, packed):
    """One stream: its order protects a block's memory once the launch that reads it is in the queue, not before."""
    N, C = 4, 16
    k, v = Made(range(N), 2 * C, 1, 128), Made(range(N), 2 * C, 1, 128)

    def call(kk, vv):
        assert k.holds(kk) and v.holds(vv)
    _pass(monkeypatch, (k, v), N, 1, C, call, packed=np.array([0, 2 * N * C], dtype=np.int32) if packed else None)
    assert k.asked.index(0) > 0                           # in the order of the steps: the rank's own block comes first


def test_blocks_made_on_demand_live_until_both_lanes_are_done(monkeypatch):
    N, C = 4, 16
    k, v = Made(range(N), 2 * C, 1, 128), Made(range(N), 2 * C, 1, 128)
    read = []

    def done():
        assert all(k.holds(a) and v.holds(b) for a, b in read)
        read.clear()
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(done))
    side = ring.SideLane(Stream(), torch.zeros(2 * C, 2, 128), torch.zeros(2, 2 * C), None, 0)
    _pass(monkeypatch, (k, v), N, 2, C, lambda kk, vv: read.append((kk, vv)), side=side)


@pytest.mark.parametrize("tensor", [False, True])
def test_only_the_blocks_that_a_pass_visits_are_asked_for(monkeypatch, tensor):
    """Documents that end with the chunk they begin in: the pruned plan reads the rank's own block and no other."""
    N, C, rank = 4, 16, 0
    cu = np.arange(0, 2 * N * C + 1, C, dtype=np.int32)
    if tensor:
        k = torch.zeros(1, 2 * C, 1, 128, dtype=torch.bfloat16)
        blocks = k, k
    else:
        blocks = Made([rank], 2 * C, 1, 128), Made([rank], 2 * C, 1, 128)
    _pass(monkeypatch, blocks, N, rank, C, lambda kk, vv: None, packed=cu)
