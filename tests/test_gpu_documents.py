"""Blocks of many documents: tiles ranked by their work, cu_seqlens searched in LDS (up to 1023 documents) and in
memory (more), against the fp64 oracle."""
import numpy as np
import pytest
import torch  # noqa: F401  (before the library: both must share torch's HIP runtime)

from paper_2408_10188_amd import binding as B
from tests.test_gpu_parity import _run_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_docs", [3, 40, 1023, 1024, 1200])
@pytest.mark.parametrize("mask", [B.MMSP_MASK_CAUSAL_DIAG, B.MMSP_MASK_FULL])
def test_many_documents(n_docs, mask):
    T = 1500
    cuts = np.sort(np.random.default_rng(n_docs).choice(np.arange(1, T), n_docs - 1, replace=False))
    cu = [0, *cuts.tolist(), T]
    _run_step(True, 4, 2, 128, T, T, dict(q_row0=0, n_q=T, k_row0=0, n_k=T, mask=mask), cu=cu, seed=n_docs)
    # a block of rows from the middle, on keys that begin and end elsewhere, with positions outside every document at either end
    _run_step(True, 3, 3, 128, 900, 1300, dict(q_row0=10, n_q=870, k_row0=5, n_k=1290, mask=mask, q_pos0=700, k_pos0=-20), cu=cu, seed=n_docs)


@pytest.mark.parametrize("cu", [[0, 63, 64, 65, 200], [0, 30, 129, 190, 200], [64, 128, 150]])
@pytest.mark.parametrize("k_pos0", [0, 10, -70])
def test_rows_that_begin_in_other_tiles_than_their_workgroup(cu, k_pos0):
    """Of 200 rows in one workgroup some see its first key tile, whose maximum is their reference, some only later ones, some none."""
    _run_step(True, 2, 1, 128, 200, 210, dict(q_row0=0, n_q=200, k_row0=0, n_k=210, mask=B.MMSP_MASK_CAUSAL_DIAG, q_pos0=0, k_pos0=k_pos0), cu=cu)


@pytest.mark.parametrize("hq,hkv", [(80, 40), (28, 14)])     # enough workgroups that tiles are ranked, by the second for dK/dV in cut ranges
@pytest.mark.parametrize("cu,q_pos0", [([0, 300, 900], 0), ([0, 620], 0), ([130, 131, 700, 1000], 90)])
@pytest.mark.parametrize("mask", [B.MMSP_MASK_CAUSAL_DIAG, B.MMSP_MASK_FULL])
def test_ranked_tiles(hq, hkv, cu, q_pos0, mask):
    _run_step(True, hq, hkv, 128, 900, 900, dict(q_row0=0, n_q=900, k_row0=0, n_k=900, mask=mask, q_pos0=q_pos0, k_pos0=q_pos0), cu=cu)
