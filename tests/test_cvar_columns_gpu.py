"""The CVaR pass with four columns of a sample's draws sorted side by side, at
the edges of its columns and groups of four, bit for bit against the float32
sums of a numpy sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("M", [129, 192, 193, 255, 257, 320, 321, 384, 385, 448, 512, 513, 1024])
def test_columns_side_by_side_bit_exact(M):
    import paper_2209_12842_amd as ra
    rng = np.random.default_rng(M)
    L = rng.gamma(2.0, 50.0, (41, M)).astype(np.float32)
    L[:20] = np.round(L[:20])                # ties
    L[1] = np.sort(L[1])                     # the tail in the last column
    L[2] = -np.sort(-L[2])                   # ... in the first
    L[3, M - 1] = np.inf
    L[4, : M - 3] = -np.inf
    L[5, 130 % M] = np.nan
    for n_tail in (1, 40, 64):
        alpha = 1.0 - (n_tail - 0.5) / M     # M - ceil(alpha M) + 1 = n_tail, half a draw from either side
        srt = -np.sort(-L, axis=1)
        ref = np.zeros(41, np.float32)
        for j in range(n_tail):
            ref = ref + srt[:, j]
        ref = ref / np.float32(n_tail)
        ref[5] = np.nan
        out = ra.cvar(torch.as_tensor(L).cuda(), alpha).cpu().numpy()
        assert np.array_equal(out, ref, equal_nan=True), n_tail
