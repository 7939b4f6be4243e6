"""Path kernel of the hierarchical layer for bf16 rows that a wave reads in one piece (padded hidden sizes of 320 to 512, and one beyond),
one round of nodes to many, in two, four and eight waves; and an infinite node weight beside lanes beyond the row."""
import numpy as np
import pytest

from test_gpu_hs_short_rows import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [257, 320, 333, 448, 512, 513])
@pytest.mark.parametrize("N,K", [(3, 4), (20, 13), (513, 4), (600, 9), (1024, 5), (1025, 5), (513, 30), (16, 60)])
def test_against_the_oracle(H, N, K):
    out, ref = run(3000, H, N, K, "bf16")
    # up to 18 terms of fp32 dot products of H products: 2^-24 of sums below 2, some hundred roundings, random signs
    assert np.max(np.abs(out - ref)) <= 2e-5


@pytest.mark.parametrize("N,K", [(6, 8), (600, 30)])
def test_an_infinite_weight(N, K):
    out, _ = run(500, 300, N, K, "bf16", spoil=True)
    gone = np.isneginf(out)                                        # one side of the root has no mass left
    assert not np.isnan(out).any() and gone.any() and not gone.all()
