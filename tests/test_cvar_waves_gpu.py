"""The CVaR of short tails (sorted inside single waves) at the edges of its
segments and columns, bit for bit against the same sums in numpy float32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


def reference(L, alpha, B):
    """Descending float32 sums of the n_tail largest scaled values of each row."""
    K, M = L.shape
    n_tail = M - min(M, max(1, int(np.ceil(float(np.float32(alpha)) * M - 1e-9)))) + 1
    if B != 1.0:
        s = np.zeros(K, np.float32)
        for j in range(M):
            s = s + L[:, j]
        mu = (s / np.float32(M))[:, None]
        # B is a power of two here, so the product is exact and the float64 sum rounds once, as an FMA does
        L = (np.float64(B) * (L - mu) + mu).astype(np.float32)
    srt = -np.sort(-L, axis=1)
    s = np.zeros(K, np.float32)
    for j in range(n_tail):
        s = s + srt[:, j]
    return s / np.float32(n_tail), n_tail


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1.0, 2.0])
@pytest.mark.parametrize("M,alpha", [(1, 0.9), (2, 0.5), (3, 0.9), (16, 0.9), (31, 0.1), (32, 0.01), (33, 0.9),
                                     (48, 0.01), (63, 0.9), (64, 0.01), (65, 0.9), (127, 0.9), (128, 0.9), (129, 0.6),
                                     (256, 0.9), (300, 0.9), (640, 0.9), (1000, 0.94),
                                     (65, 0.01), (128, 0.5)])  # the last two: tails longer than a wave
def test_short_tails_bit_exact(M, alpha, B):
    import paper_2209_12842_amd as ra
    rng = np.random.default_rng(M)
    K = 77
    L = rng.gamma(2.0, 50.0, (K, M)).astype(np.float32)
    L[: K // 2] = np.round(L[: K // 2])  # ties
    L[0] = 7.0
    ref, n_tail = reference(L, alpha, B)
    out = ra.cvar(torch.as_tensor(L).cuda(), alpha, B).cpu().numpy()
    assert np.array_equal(out, ref), (n_tail, np.abs(out - ref).max())


@pytest.mark.gpu
@pytest.mark.parametrize("M", [16, 48, 64, 100, 300])
def test_infinite_and_undefined_costs(M):
    import paper_2209_12842_amd as ra
    rng = np.random.default_rng(M)
    L = rng.gamma(2.0, 50.0, (12, M)).astype(np.float32)
    L[1, M // 2] = np.inf
    L[2, 0] = -np.inf
    L[3, M - 1] = np.nan
    L[4] = -np.inf
    ref, _ = reference(L, 0.9, 1.0)
    ref[3] = np.nan
    out = ra.cvar(torch.as_tensor(L).cuda(), 0.9).cpu().numpy()
    assert np.array_equal(out, ref, equal_nan=True)


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1.0, 2.0])
@pytest.mark.parametrize("M,alpha", [(3, 0.01), (4, 0.01), (5, 0.01), (5, 0.9), (40, 0.5), (47, 0.9), (48, 0.76), (48, 0.73), (52, 0.55),
                                     (54, 0.45), (55, 0.42), (55, 0.4), (64, 0.52), (64, 0.48), (65, 0.25), (65, 0.2)])
def test_either_side_of_the_pass_rule(M, alpha, B):
    """Bits at the sizes where the entry point changes from one pass to the
    other; a cost that is not a number makes its sample's CVaR one in both."""
    import paper_2209_12842_amd as ra
    rng = np.random.default_rng(M)
    L = rng.gamma(2.0, 50.0, (531, M)).astype(np.float32)
    L[:200] = np.round(L[:200])
    undefined = {7: 0, 8: M // 2, 530: M - 1}
    ref, n_tail = reference(L, alpha, B)
    for k, m in undefined.items():
        L[k, m] = np.nan
        ref[k] = np.nan
    out = ra.cvar(torch.as_tensor(L).cuda(), alpha, B).cpu().numpy()
    assert np.array_equal(out, ref, equal_nan=True), n_tail
