"""The fp32 kernels against the fp64 oracle at the edges of their 16-row blocks, and with values that are
not finite in rows no query sees."""
import math

import numpy as np
import pytest
import torch

from paper_2408_10188_amd import binding as B
from paper_2408_10188_amd import ring
from tests.helpers import DEV, max_abs, to_dev, to_host64
from oracle import mmsp_oracle as orc

pytestmark = pytest.mark.gpu


def _step(d, hq, hkv, n_q, n_k, mask, q_pos0, cu, spoil):
    rng = np.random.default_rng(1000 * n_q + n_k)
    q, k, v, do = (rng.standard_normal(s, dtype=np.float32) for s in ((n_q, hq, d), (n_k, hkv, d), (n_k, hkv, d), (n_q, hq, d)))
    scale = 1 / math.sqrt(d)
    blk = dict(q_row0=0, n_q=n_q, k_row0=0, n_k=n_k, q_pos0=q_pos0, k_pos0=0, mask=mask)
    q64, k64, v64, do64 = (x.astype(np.float64) for x in (q, k, v, do))
    o_ref, l_ref = orc.step_fwd(q64, k64, v64, blk, scale, cu)
    delta = orc.delta(do64, o_ref)
    ref = orc.step_bwd(q64, k64, v64, do64, l_ref, delta, blk, scale, cu)
    seen_k = np.zeros(n_k, dtype=bool)
    for i in range(n_q):
        p = q_pos0 + i
        vis = np.arange(n_k) <= p if mask == B.MMSP_MASK_CAUSAL_DIAG else np.ones(n_k, dtype=bool)
        if cu is not None:
            doc = np.searchsorted(cu, np.arange(n_k), side="right")
            own = np.searchsorted(cu, p, side="right")
            vis &= (doc == own) & (cu[0] <= p < cu[-1])
        seen_k |= vis
    if spoil:                       # rows that no query sees may hold anything
        k[~seen_k], v[~seen_k] = np.nan, np.inf
    qd, kd, vd, dod = (to_dev(x, False) for x in (q, k, v, do))
    shape = ring.shape_for(qd, kd, B.MMSP_F32, n_q, scale)
    cud = None if cu is None else torch.tensor(cu, dtype=torch.int32, device=DEV)
    block = B.make_block(0, n_q, 0, n_k, mask, q_pos0, 0, cud, 0 if cu is None else len(cu) - 1)
    o, lse = (torch.full(s, math.nan, device=DEV) for s in ((n_q, hq, d), (hq, n_q)))
    B.mmsp_attn_step_fwd(shape, block, qd, kd, vd, o, lse, False)
    dq = torch.zeros_like(o)
    dk, dv = torch.full_like(kd, math.nan), torch.full_like(vd, math.nan)
    lref, dref = (to_dev(x, False) for x in (l_ref, delta))
    B.mmsp_attn_step_bwd(shape, block, qd, kd, vd, None, dod, lref, dref, False, dq, dk, dv, False)
    for got, want in zip((o, lse, dq, dk, dv), (o_ref, l_ref, *ref)):
        # a sum of n fp32 terms of either sign rounds by about sqrt(n) * 2^-24 of its largest term: below 1e-5 of the largest
        # result for the few hundred terms here
        largest = max(1.0, float(np.abs(want[np.isfinite(want)]).max(initial=0)))
        assert max_abs(to_host64(got), want) <= 1e-5 * largest
    B.mmsp_attn_step_fwd(shape, block, qd, kd, vd, o, lse, True)          # the same block once more: the sums double, O stays
    assert max_abs(to_host64(o), o_ref) <= 1e-5 * max(1.0, float(np.abs(o_ref).max(initial=0)))
    assert max_abs(to_host64(lse), l_ref + math.log(2.0)) <= 1e-5 * 10


@pytest.mark.parametrize("d,hq,hkv", [(64, 2, 1), (128, 4, 2), (128, 3, 3)])
@pytest.mark.parametrize("n_q,n_k,q_pos0", [(1, 1, 0), (15, 17, 2), (16, 128, 112), (33, 129, 60), (130, 300, 170)])
@pytest.mark.parametrize("masked", ["full", "causal", "documents"])
def test_f32_step_at_block_edges(d, hq, hkv, n_q, n_k, q_pos0, masked):
    cu = [0, max(1, n_k // 3), max(2, n_k // 2 + 1), n_k + n_q + q_pos0] if masked == "documents" else None
    mask = B.MMSP_MASK_FULL if masked == "full" else B.MMSP_MASK_CAUSAL_DIAG
    for spoil in (False, True):
        _step(d, hq, hkv, n_q, n_k, mask, q_pos0, cu, spoil)
