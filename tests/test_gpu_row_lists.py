"""Forward and backward steps at the edges of the kernels' tiles and of the rules that share them out, against the fp64 oracle.  The rows of the heads that share
a KV head are one list cut into tiles of 128 or 256 (row, head) pairs, so an edge can fall between two heads of a row;
the key loop takes four tiles of 64 per trip and starts in the middle of one."""
import pytest
import torch  # noqa: F401  loads the HIP runtime that the library shares

from paper_2408_10188_amd import binding as B
from tests.test_gpu_parity import _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,n_q", [
    (14, 2, 1), (14, 2, 18), (14, 2, 19), (14, 2, 37),       # 7, 126, 133, 259 pairs per KV head
    (6, 2, 43), (6, 2, 86),                                  # 129, 258
    (12, 1, 32), (5, 5, 128), (5, 5, 129),                   # 384; groups of one, without the head-to-XCD mapping
    (28, 4, 1190),                                           # 132 workgroups of 256 pairs
])
@pytest.mark.parametrize("n_k", [1, 64, 65, 130, 200, 257])
def test_tiles_of_the_row_list(hq, hkv, n_q, n_k):
    for mask, pos in ((B.MMSP_MASK_FULL, 0), (B.MMSP_MASK_CAUSAL_DIAG, n_k - n_q)):
        _run_step(True, hq, hkv, 128, n_q + 5, n_k + 3, dict(q_row0=2, n_q=n_q, k_row0=1, n_k=n_k, mask=mask, q_pos0=pos, k_pos0=0), seed=n_q + n_k)


@pytest.mark.parametrize("hq,hkv", [(14, 2), (3, 3)])
@pytest.mark.parametrize("cu", [[0, 5, 70, 71, 200, 330], [0, 330], [100, 130, 250]])
def test_documents_shorter_than_a_tile(hq, hkv, cu):
    for mask in (B.MMSP_MASK_FULL, B.MMSP_MASK_CAUSAL_DIAG):
        _run_step(True, hq, hkv, 128, 330, 330, dict(q_row0=0, n_q=330, k_row0=0, n_k=330, mask=mask, q_pos0=0, k_pos0=0), cu=cu, seed=len(cu))


@pytest.mark.parametrize("hq,hkv,n_q,n_k,mask,pos", [
    (7, 1, 1300, 130, B.MMSP_MASK_FULL, 0),                  # 147 elements a key tile, dealt to 32 workgroups
    (7, 1, 1100, 1100, B.MMSP_MASK_CAUSAL_DIAG, 0),
    (5, 5, 70, 900, B.MMSP_MASK_CAUSAL_DIAG, 830),           # two elements: not dealt out
    (4, 2, 200, 129, B.MMSP_MASK_CAUSAL_DIAG, -20),          # one live key in the last tile, rows that see nothing
])
def test_shares_of_a_key_tile(hq, hkv, n_q, n_k, mask, pos):
    _run_step(True, hq, hkv, 128, n_q + 1, n_k + 2, dict(q_row0=1, n_q=n_q, k_row0=2, n_k=n_k, mask=mask, q_pos0=pos, k_pos0=0), seed=n_q)


@pytest.mark.parametrize("q_pos0", [98, 99, 100, 5000])
def test_a_causal_mask_that_hides_nothing(q_pos0):
    """From q_pos0 = 99 on no key of 0..99 follows the first query: such a block runs as one without a mask."""
    _run_step(True, 6, 2, 128, 64, 100, dict(q_row0=0, n_q=64, k_row0=0, n_k=100, mask=B.MMSP_MASK_CAUSAL_DIAG, q_pos0=q_pos0, k_pos0=0), seed=q_pos0)


@pytest.mark.parametrize("hq,hkv,n_q,n_k", [
    (2, 1, 37, 41), (8, 2, 399, 401),                        # dK and dV apart: 3 + 3 + 6 workgroups; 52 + 52 + 200, more than 256 in all
    (8, 8, 120, 250),                                        # one launch, dK and dV together: 128 + 64
    (8, 8, 257, 259),                                        # two launches: 136, 136
])
@pytest.mark.parametrize("d", [64, 128])
def test_gradients_in_fp32_by_launches(hq, hkv, n_q, n_k, d):
    for mask, pos, cu in ((B.MMSP_MASK_FULL, 0, None), (B.MMSP_MASK_CAUSAL_DIAG, n_k - n_q - 20, None), (B.MMSP_MASK_CAUSAL_DIAG, 0, [0, 3, 20, n_q])):
        _run_step(False, hq, hkv, d, n_q + 2, n_k + 3, dict(q_row0=0, n_q=n_q, k_row0=0, n_k=n_k, mask=mask, q_pos0=pos, k_pos0=0), cu=cu, seed=n_q + d)
