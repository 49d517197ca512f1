"""Matrix-core sweeps whose blocks take several splits one after another: an odd number of one-tile splits
(the last run is short), a ragged last tile, both chains of the column sweep; bounds as derived in
test_gpu_lamp.py."""
from __future__ import annotations

import pytest
import torch

from tests.test_gpu_lamp import _mfma_step_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,dtype,shape", [("bf16_mfma", torch.bfloat16, (2060, 4000, 3)),
                                              ("fp16x3_mfma", None, (2060, 3990, 20))])
def test_step_with_runs_of_splits(form, dtype, shape):
    _mfma_step_check(form, dtype, shape)
