"""The host loop of ring.py by itself: which rows its calls leave how, and what it holds while they run.  The calls of the library are
replaced by recorders, so no GPU is needed; layouts and plans are the library's own."""
import types

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
