"""A query row whose scores hold a NaN ends as a row of NaNs: no merge on the way (of ring steps, of launch lanes, of
key ranges, of an fp32 workgroup's wavefronts) may replace it by what other keys contribute, or by zeros."""
import math

import pytest
import torch

from paper_2408_10188_amd import binding as B
from paper_2408_10188_amd import ring
from tests.helpers import DEV, RankProblem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("lanes,fused", [(1, True), (1, False), (2, True)])
@pytest.mark.parametrize("rank", [0, 1])
@pytest.mark.parametrize("where", ["query", "key"])
def test_ring_keeps_nan_rows(dtype, d, lanes, fused, rank, where):
    C, row, key = 96, 100, 130
    prob = RankProblem(dict(dtype=dtype, Hq=4, Hkv=2, d=d, N=2, C=C, sigma=0.5, seed=2))
    q, _ = prob.rank_inputs(rank)
    want = torch.zeros(2 * C, 4, dtype=torch.bool, device=DEV)
    if where == "query":
        q[row, 1] = math.nan
        want[row, 1] = True
    else:                                                   # a key of the rank's own block: every later row of its two heads sees it
        prob.k_zz[rank, key, 1, 7] = math.nan
        want[key:, 2:] = True
    out = prob.run_gpu(rank, q, fused_merge=fused, two_streams=lanes == 2)
    for o in (out["o_acc"], out["o_final"]):
        assert torch.equal(torch.isnan(o).any(2), want)
        assert torch.equal(torch.isnan(o).all(2), want)
