"""Rules of the GEMM plans, on the host."""
import pytest

from tests._plans import gemm_plan_shared

CUS = 256


@pytest.mark.parametrize("d", list(range(2176, 8193, 128)))
def test_shared_projection_waves(d):
    """Context and block rows in one launch above the short K: the waves and the K split that fill
    one round of workgroups best, ties to fewer splits and then to more waves, each split of 8 K
    steps at least; 8 waves alone for K above 4096."""
    for rows, M in ((2, 1), (33, 16), (128, 64), (129, 128), (160, 32), (192, 64), (256, 128)):
        def score(nw, s):
            tiles = -(-rows // 128) * -(-2 * d // (32 * nw)) + -(-d // (32 * nw))
            rounds = -(-tiles * s // CUS)
            return round(tiles * s / (rounds * CUS) / rounds + (rounds == 1), 9)
        nw, splits = max(((nw, s) for nw in ((4, 8) if d <= 4096 else (8,)) for s in range(1, 17)
                          if s == 1 or d // 64 // s >= 8), key=lambda x: (score(*x), -x[1], x[0]))
        p = gemm_plan_shared(rows, 2 * d, M, d, d)
        assert (p.nw, p.splits, p.tn, p.nt) == (nw, splits, 1, False), (rows, M)


@pytest.mark.parametrize("d", [256, 1024, 2048])
def test_shared_projection_of_short_k_takes_four_waves(d):
    for rows, M in ((2, 1), (128, 64), (256, 128)):
        p = gemm_plan_shared(rows, 2 * d, M, d, d)
        assert (p.nw, p.tn, p.nt) == (4, 1, False)
