"""The binary64 product on each of its tiles at the edges of tiles and of its look-ahead: reductions of less than one 16-deep tile up to several with and without a
rest, rows and columns that end inside a tile, the four transposes.  Against numpy; a row of infinities at the edge stays in that row."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_tiles(nqopt, tile, ta, tb):
    import torch
    nqopt.set("dgemm_tile", tile)
    for M, N, K in [(1, 1, 1), (3, 130, 15), (129, 65, 16), (127, 127, 17), (128, 64, 31), (64, 200, 32), (257, 3, 33), (130, 129, 48), (70, 66, 63), (128, 128, 64),
                    (200, 100, 79), (65, 129, 80), (140, 190, 96), (128, 260, 113)]:
        g = np.random.default_rng(M * 7 + N * 3 + K)
        a, b = g.standard_normal((M, K)), g.standard_normal((K, N))
        if M > 1:
            a[M - 1] = np.inf
        out = torch.full((M, N + 1), float("nan"), dtype=torch.float64, device="cuda")
        nq.nq_dgemm(ta, tb, M, N, K, 1.0, dev(a.T if ta else a), M if ta else K, dev(b.T if tb else b), K if tb else N, 0.0, out, N + 1)
        got = out.cpu().numpy()
        ref = a[: max(1, M - 1)] @ b
        # K products and additions, each rounded to 2^-53 of partial sums that stay below the sum of magnitudes
        bound = (K + 4) * 2.0 ** -53 * (np.abs(a[: max(1, M - 1)]) @ np.abs(b)).max()
        assert np.abs(got[: max(1, M - 1), :N] - ref).max() <= bound, (M, N, K)
        assert np.isnan(got[:, N]).all()                     # nothing beyond the columns is touched
        if M > 1:
            assert not np.isfinite(got[M - 1, :N]).any()
