"""Matrix-core sweeps whose blocks take several splits one after another: an odd number of one-tile splits
(the last run is short), a ragged last tile, both chains of the column sweep; bounds as derived in
test_gpu_lamp.py."""
from __future__ import annotations

import pytest
import torch

from tests import test_gpu_dims as dims
from tests.test_gpu_lamp import _mfma_step_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,dtype,shape", [("bf16_mfma", torch.bfloat16, (2060, 4000, 3)),
                                              ("fp16x3_mfma", None, (2060, 3990, 20))])
def test_step_with_runs_of_splits(form, dtype, shape):
    _mfma_step_check(form, dtype, shape)


@pytest.mark.parametrize("n,m,d", [(1100, 1000, 40), (640, 20000, 20), (20000, 650, 17)])
def test_fp64_product_step_with_runs_of_splits(n, m, d):
    """The FP64 products (d > 16): runs of one-tile splits with a short last one, and splits of three tiles
    (the carry of every second tile starts again with each split); bounds of test_gpu_dims.py."""
    dims.test_step_matches_oracle(n, m, d, "sqeuclid")
