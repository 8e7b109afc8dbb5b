"""The choice of a product's kernel, on the host: bounds that a kernel needs."""
import os

import pytest

torch = pytest.importorskip("torch")
from paper_2607_24841_amd import binding as B  # noqa: E402

from ._plan import plan  # noqa: E402

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libnmdlm.so not built")


@pytest.mark.parametrize("T,M,K,N", [(3, 1008, 64, 8 << 20), (3, 174000, 64, 33200), (5, 80, 64, 3 << 23),
                                     (7, 1000, 1, 3 << 20)])
def test_lean_grids_stay_below_the_float_quotient(T, M, K, N):
    """The lean product takes its tile's column as a float quotient, exact for
    fewer than 2^21 tiles (test_div_small); larger grids divide in integers."""
    p = plan(T, M, K, N, blocked=1)
    assert p.status == B.NMDLM_OK
    assert ((N + 63) // 64) * p.row_blocks >= 1 << 21
    assert p.kernel == "words"
    half = plan(T, M, K, N // 8, blocked=1)            # under the bound: lean again
    assert ((N // 8 + 63) // 64) * half.row_blocks < 1 << 21
    assert half.kernel == "lean"
