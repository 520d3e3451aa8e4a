"""Forward and dQ steps whose key range is cut into several workgroups per query tile (few query rows on many
keys), against the fp64 oracle: ranges that do not divide the tiles, masks that leave ranges empty, and every
amount of workspace, whose end no kernel may pass."""
import math

import numpy as np
import pytest
import torch

from oracle import mmsp_oracle as orc
from paper_2408_10188_amd import binding as B
from paper_2408_10188_amd import ring, synth
from tests.helpers import DEV, NORTH_STAR_TOL, max_abs, to_dev, to_host64
from tests.test_gpu_parity import _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv", [(7, 1), (6, 3)])       # with and without the head-to-XCD mapping
@pytest.mark.parametrize("n_q,n_k,mask,cu", [
    (1, 1500, B.MMSP_MASK_FULL, None),
    (203, 2049, B.MMSP_MASK_CAUSAL_DIAG, None),
    (257, 1984, B.MMSP_MASK_CAUSAL_DIAG, None),
    (300, 2500, B.MMSP_MASK_CAUSAL_DIAG, [0, 900, 2301, 2302, 2480, 2500]),   # rows of several documents: most ranges empty
    (300, 2500, B.MMSP_MASK_FULL, [0, 2301, 2450]),                           # the last rows lie in no document
])
def test_few_rows_on_many_keys(hq, hkv, n_q, n_k, mask, cu):
    _run_step(True, hq, hkv, 128, n_q + 9, n_k + 70, dict(q_row0=4, n_q=n_q, k_row0=33, n_k=n_k, mask=mask, q_pos0=n_k - n_q, k_pos0=0),
              cu=cu, seed=n_q + n_k)


@pytest.mark.parametrize("ranges", [0, 1, 2.01, 3, 40])
@pytest.mark.parametrize("accumulate", [False, True])
def test_workspace_of_any_size(ranges, accumulate):
    hq, hkv, d, n_q, n_k, scale = 4, 2, 128, 77, 2000, 1 / math.sqrt(128)
    rng = np.random.default_rng(5)
    q, k, v = (synth.bf16_round(rng.standard_normal(s, dtype=np.float32) * 0.5) for s in ((n_q, hq, d), (n_k, hkv, d), (n_k, hkv, d)))
    blk = dict(q_row0=0, n_q=n_q, k_row0=0, n_k=n_k, q_pos0=n_k - n_q, k_pos0=0, mask=B.MMSP_MASK_CAUSAL_DIAG)
    o_ref, l_ref = orc.step_fwd(*(x.astype(np.float64) for x in (q, k, v)), blk, scale, None)
    qd, kd, vd = (to_dev(x, True) for x in (q, k, v))
    shape = ring.shape_for(qd, kd, B.MMSP_BF16, n_q, scale)
    block = B.make_block(0, n_q, 0, n_k, blk["mask"], blk["q_pos0"], 0)
    given = int(ranges * n_q * hq * 129 * 4)
    ws = torch.full((given + 4096,), 77, dtype=torch.uint8, device=DEV)
    # accumulate: onto the result of the same keys, so that O stays and every sum doubles
    o = to_dev(o_ref.astype(np.float32), False) if accumulate else torch.full((n_q, hq, d), math.nan, device=DEV)
    lse = to_dev(l_ref.astype(np.float32), False) if accumulate else torch.full((hq, n_q), math.nan, device=DEV)
    B.mmsp_attn_step_fwd(shape, block, qd, kd, vd, o, lse, accumulate, ws, given)
    assert max_abs(to_host64(o), o_ref) <= NORTH_STAR_TOL["bf16"]["o"]
    assert max_abs(to_host64(lse), l_ref + (math.log(2.0) if accumulate else 0.0)) <= NORTH_STAR_TOL["bf16"]["lse"]
    assert bool((ws[given:] == 77).all())
    assert bool((ws == 77).all()) == (ranges < 2)         # with room for two ranges the keys are cut


@pytest.mark.parametrize("gradients", ["dq", "all"])
@pytest.mark.parametrize("n_q,n_k", [(77, 2000), (300, 1984)])
def test_dq_ranges_stay_in_the_workspace(gradients, n_q, n_k):
    hq, hkv, d, scale = 4, 2, 128, 1 / math.sqrt(128)
    rng = np.random.default_rng(6)
    q, k, v = (synth.bf16_round(rng.standard_normal(s, dtype=np.float32) * 0.5) for s in ((n_q, hq, d), (n_k, hkv, d), (n_k, hkv, d)))
    do = synth.bf16_round(rng.standard_normal((n_q, hq, d), dtype=np.float32))
    blk = dict(q_row0=0, n_q=n_q, k_row0=0, n_k=n_k, q_pos0=n_k - n_q, k_pos0=0, mask=B.MMSP_MASK_CAUSAL_DIAG)
    q64, k64, v64, do64 = (x.astype(np.float64) for x in (q, k, v, do))
    o_ref, l_ref = orc.step_fwd(q64, k64, v64, blk, scale, None)
    delta = orc.delta(do64, o_ref)
    ref = orc.step_bwd(q64, k64, v64, do64, l_ref, delta, blk, scale, None)
    qd, kd, vd, dod = (to_dev(x, True) for x in (q, k, v, do))
    lse, dl = (to_dev(x.astype(np.float32), False) for x in (l_ref, delta))
    shape = ring.shape_for(qd, kd, B.MMSP_BF16, n_q, scale)
    given = B.mmsp_workspace_bytes(shape, n_q, n_k, True)
    ws = torch.full((given + 4096,), 77, dtype=torch.uint8, device=DEV)
    dq = torch.zeros(n_q, hq, d, device=DEV)
    dk, dv = (torch.full((n_k, hkv, d), math.nan, device=DEV) for _ in range(2))
    both = gradients == "all"
    B.mmsp_attn_step_bwd(shape, B.make_block(0, n_q, 0, n_k, blk["mask"], blk["q_pos0"], 0), qd, kd, vd, None, dod, lse, dl, False, dq,
                         dk if both else None, dv if both else None, False, ws, given)
    for got, want in zip((dq, dk, dv) if both else (dq,), ref):
        assert max_abs(to_host64(got), want) <= NORTH_STAR_TOL["bf16"]["g"]
    assert bool((ws[given:] == 77).all())
    stats = 2 * hq * 4 * ((n_q + 63) // 64 * 64)          # row statistics, written for dK/dV only; the partial results lie behind them
    assert bool((ws[:stats] == 77).all()) != both
    assert bool((ws[stats:stats + 2 * n_q * hq * d * 4] != 77).any())


def test_a_row_of_nans_stays_one():
    hq, hkv, n_q, n_k = 2, 1, 40, 3000
    gen = torch.Generator(device=DEV).manual_seed(1)
    q, k, v = (torch.randn(s, device=DEV, generator=gen).bfloat16() for s in ((n_q, hq, 128), (n_k, hkv, 128), (n_k, hkv, 128)))
    q[7, 1] = math.nan
    shape = ring.shape_for(q, k, B.MMSP_BF16, n_q)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    o, lse = torch.zeros(n_q, hq, 128, device=DEV), torch.zeros(hq, n_q, device=DEV)
    B.mmsp_attn_step_fwd(shape, B.make_block(0, n_q, 0, n_k, B.MMSP_MASK_FULL), q, k, v, o, lse, False, ws, ws.numel())
    nan = torch.isnan(o).all(2)
    assert bool(nan[7, 1]) and int(torch.isnan(o).any(2).sum()) == 1


@pytest.mark.parametrize("docs,cut", [(1, True), (4, True), (150, False)])
def test_short_documents_are_not_cut(docs, cut):
    """The host knows the documents' number only; with many of them a row sees few keys and ranges would be empty."""
    hq, n_q, n_k = 8, 100, 6000
    gen = torch.Generator(device=DEV).manual_seed(3)
    q, k, v = (torch.randn(s, device=DEV, generator=gen).bfloat16() for s in ((n_q, hq, 128), (n_k, 1, 128), (n_k, 1, 128)))
    cu = torch.linspace(0, n_k, docs + 1, device=DEV).to(torch.int32)
    shape = ring.shape_for(q, k, B.MMSP_BF16, n_q)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    o, lse = torch.zeros(n_q, hq, 128, device=DEV), torch.zeros(hq, n_q, device=DEV)
    B.mmsp_attn_step_fwd(shape, B.make_block(0, n_q, 0, n_k, B.MMSP_MASK_CAUSAL_DIAG, n_k - n_q, 0, cu, docs), q, k, v, o, lse, False, ws, ws.numel())
    assert bool(ws.any()) == cut
