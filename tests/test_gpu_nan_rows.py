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


@pytest.mark.parametrize("d", [64, 128])
def test_f32_wavefront_without_weight_keeps_its_nan(d):
    """Keys 0 to 15, one wavefront's share, lie 200 below all others, so that its weight in the merge is exp(-200) = 0."""
    n_q, n_k, key = 20, 128, 3
    q, k, v = (torch.zeros(n, 1, d, device=DEV) for n in (n_q, n_k, n_k))
    q[:, 0, 0], k[:16, 0, 0], v[:] = math.sqrt(d), -200.0, 1.0
    k[key, 0, 1] = math.nan
    shape = ring.shape_for(q, k, B.MMSP_F32, n_q)
    o, lse = torch.zeros(n_q, 1, d, device=DEV), torch.zeros(1, n_q, device=DEV)
    B.mmsp_attn_step_fwd(shape, B.make_block(0, n_q, 0, n_k, B.MMSP_MASK_FULL), q, k, v, o, lse, False)
    assert bool(torch.isnan(o).all()) and bool((lse == -math.inf).all())
