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


@pytest.mark.parametrize("running", [None, -math.inf, 1.0])       # overwrite / merge into an empty and into a full running result
@pytest.mark.parametrize("where", ["query", "key"])
def test_key_ranges_report_nan_rows_as_one_workgroup_does(running, where):
    hq, n_q, n_k = 2, 40, 3000
    gen = torch.Generator(device=DEV).manual_seed(1)
    q, k, v = (torch.randn(s, device=DEV, generator=gen).bfloat16() for s in ((n_q, hq, 128), (n_k, 1, 128), (n_k, 1, 128)))
    if where == "query":
        q[7, 1] = math.nan
    else:
        k[n_k - 20, 0, 3] = math.nan                              # the rows from the 20th on see it
    shape = ring.shape_for(q, k, B.MMSP_BF16, n_q)
    block = B.make_block(0, n_q, 0, n_k, B.MMSP_MASK_CAUSAL_DIAG, n_k - n_q, 0)
    got = []
    for room in (0, 64 << 20):                                    # one workgroup for all keys, then several
        ws = torch.zeros(room + 16, dtype=torch.uint8, device=DEV)
        o, lse = torch.full((n_q, hq, 128), 0.25, device=DEV), torch.full((hq, n_q), 0.0 if running is None else running, device=DEV)
        B.mmsp_attn_step_fwd(shape, block, q, k, v, o, lse, running is not None, ws, room)
        assert (room > 0) == bool(ws.any())                       # the partial results were kept there
        got.append((o, lse))
    (o1, lse1), (o2, lse2) = got
    assert torch.equal(torch.isnan(o1), torch.isnan(o2)) and (bool(torch.isnan(o1).any()) or running == -math.inf)
    assert torch.equal(torch.isfinite(lse1), torch.isfinite(lse2))
    # two bf16 roundings of P against different references: 2^-8 of a mean of unit values, over many keys
    torch.testing.assert_close(o1.nan_to_num(), o2.nan_to_num(), atol=2e-2, rtol=0)
    torch.testing.assert_close(lse1, lse2, atol=1e-3, rtol=0)
