"""The two-stage aggregation kernel's stage-1 mean by a reciprocal, exact (CPU)."""
import numpy as np

NMAX = (2 * 17 + 1) ** 2


def test_mean_by_reciprocal_and_remainder():
    """The two-stage kernel's stage-1 mean floor((S + floor(N/2)) / N): q =
    trunc(fma((float)S, RN(1/N), 0.25)) is that or one less, and the remainder
    S - q N >= ceil(N/2) tells which, for every N <= 1225 and S <= N 2^20
    (0.25 plus less than 0.19 of rounding stays below 1 - (N - 1 - N/2) / N).
    Checked at the rounding boundaries of many quotients, the largest among
    them; the product of two floats plus 0.25 is exact in a double here or
    rounds far below what decides."""
    rng = np.random.default_rng(11)
    for N in range(1, NMAX + 1):
        k = np.unique(np.concatenate([np.array([0, 1, 2, (1 << 20) - 1, 1 << 20]),
                                      rng.integers(0, 1 << 20, 400)])).astype(np.int64)
        h = N // 2
        S = np.concatenate([k * N + o for o in (-h - 1, -h, -1, 0, 1, N - h - 1, N - h)])
        S = S[(S >= 0) & (S <= N << 20)]
        want = (S + h) // N
        rcp = np.float32(1.0) / np.float32(N)
        t = S.astype(np.float32).astype(np.float64) * np.float64(rcp) + 0.25
        q = t.astype(np.float32).astype(np.int64)
        assert ((q == want) | (q == want - 1)).all(), N
        assert np.array_equal(q + (S - q * N >= (N + 1) // 2), want), N
        assert (np.abs(S - q * N) < 1 << 31).all() and (q < 1 << 23).all()
