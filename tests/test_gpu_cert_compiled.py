"""The certificate's pair passes with 32 and 64 coordinates in registers, and at 64 the change to the run-time
form below 61440 own points (in rows and in columns), by the same comparison as the others."""
from __future__ import annotations

import pytest

from tests.test_gpu_certpass import test_certificate_passes as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,d", [(1, 9, 32), (70, 263, 32), (300, 7, 32), (61440, 9, 64), (61439, 17, 64), (9, 62001, 64)])
def test_wide_points_in_registers(n, m, d):
    check(n, m, d, "sqeuclid")
