"""dK and dV of blocks that add to what is there, and of key tiles whose shares take turns over the XCDs of a KV head."""
import pytest
import torch

from paper_2408_10188_amd import binding as B
from paper_2408_10188_amd import ring
from tests.test_gpu_parity import DEV, _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,n_q,n_k,mask,pos,exact", [
    (4, 2, 33, 1, B.MMSP_MASK_FULL, 0, True), (4, 2, 64, 129, B.MMSP_MASK_FULL, 0, True), (8, 8, 50, 31, B.MMSP_MASK_FULL, 0, True),
    (5, 5, 70, 900, B.MMSP_MASK_CAUSAL_DIAG, 830, True), (4, 2, 20, 160, B.MMSP_MASK_CAUSAL_DIAG, -3, True),   # keys that no row sees keep what they have
    (28, 4, 120, 97, B.MMSP_MASK_CAUSAL_DIAG, 0, False),     # several shares: the reduction adds, after summing onto what is there
])
def test_adding_leaves_the_sum(hq, hkv, n_q, n_k, mask, pos, exact):
    g = torch.Generator(device=DEV)
    g.manual_seed(n_q + n_k)
    rnd = lambda *s: torch.randn(*s, device=DEV, generator=g)
    q, do = (rnd(n_q, hq, 128).bfloat16() for _ in range(2))
    k, v = (rnd(n_k + 5, hkv, 128).bfloat16() for _ in range(2))
    lse, delta = rnd(hq, n_q) * .1 + 5., rnd(hq, n_q)
    shape = ring.shape_for(q, k, B.MMSP_BF16, n_q)
    blk = B.make_block(0, n_q, 3, n_k, mask, pos, 0)
    nb = B.mmsp_workspace_bytes(shape, n_q, n_k, True)
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
    base = [rnd(n_k + 5, hkv, 128) for _ in range(2)]
    plain, added = [torch.zeros_like(b) for b in base], [b.clone() for b in base]
    B.mmsp_attn_step_bwd(shape, blk, q, k, v, None, do, lse, delta, False, None, *plain, False, ws, nb)
    B.mmsp_attn_step_bwd(shape, blk, q, k, v, None, do, lse, delta, False, None, *added, True, ws, nb)
    torch.cuda.synchronize()
    assert plain[0].abs().max() > 0 and plain[1].abs().max() > 0
    for b, p, a in zip(base, plain, added):
        if exact:
            assert torch.equal(a, b + p)                  # one fp32 addition per element, rows 0..2 and the last two plus zero
        else:                                             # shares and what is there are summed in another order: fewer than 40 roundings of 2^-24
            assert ((a - (b + p)).abs() <= 40 * 2. ** -24 * (b.abs() + 8 * p.abs().max())).all()


@pytest.mark.parametrize("hq,hkv,n_q,n_k", [
    (28, 4, 200, 390), (14, 2, 260, 390), (4, 2, 500, 700), (7, 1, 300, 650), (2, 1, 900, 257),   # two, four and eight XCDs a KV head
])
def test_shares_that_take_turns(hq, hkv, n_q, n_k):
    for mask, pos, cu in ((B.MMSP_MASK_FULL, 0, None), (B.MMSP_MASK_CAUSAL_DIAG, max(0, n_k - n_q), None), (B.MMSP_MASK_CAUSAL_DIAG, 0, [0, 90, 100, max(n_q, n_k)])):
        _run_step(True, hq, hkv, 128, n_q, n_k + 2, dict(q_row0=0, n_q=n_q, k_row0=1, n_k=n_k, mask=mask, q_pos0=pos, k_pos0=0), cu=cu, seed=n_q)
