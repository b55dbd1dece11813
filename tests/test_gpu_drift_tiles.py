"""ress_block_drift_sq at the edges of its 16-token tiles and of its waves' shares
of a block, with a Gram matrix that is not symmetric (the kernel folds M's
off-diagonal blocks), against x^T M x in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bq", [64, 128])
@pytest.mark.parametrize("N", [1, 15, 16, 17, 63, 65, 127, 129, 200, 321])
def test_drift_tile_edges(N, bq):
    import torch

    import paper_2609_35593_amd as ress

    H = 2
    rng = np.random.default_rng(1000 * bq + N)
    a = rng.standard_normal((H, N, 64)).astype(np.float32)
    b = rng.standard_normal((H, N, 64)).astype(np.float32)
    gram = rng.standard_normal((H, 64, 64)).astype(np.float32)
    got = ress.ress_block_drift_sq(*(torch.from_numpy(t).cuda() for t in (a, b, gram)), bq=bq).cpu().numpy()
    x = a.astype(np.float64) - b.astype(np.float64)
    # Each term is a product of exact float64 values; a sum of n <= 128 * 64^2 of them in any order differs from
    # another by at most n 2^-52 times the sum of their magnitudes, and by about sqrt(n) 2^-53 in practice: 2^-40
    # bounds it with room.
    for i in range(got.shape[1]):
        xs = x[:, i * bq:(i + 1) * bq]
        ref = np.einsum("htc,hcd,htd->h", xs, gram.astype(np.float64), xs)
        mag = np.einsum("htc,hcd,htd->h", np.abs(xs), np.abs(gram).astype(np.float64), np.abs(xs))
        assert np.all(np.abs(got[:, i] - ref) <= 2.0 ** -40 * mag)


@pytest.mark.parametrize("N", [16, 17, 70, 128, 130])
def test_drift_infinite_gram(N):
    """A Gram matrix with an infinite diagonal entry gives an infinite result in every block, ragged ones too: the
    rows that pad a block's last tile have no part in it."""
    import torch

    import paper_2609_35593_amd as ress

    rng = np.random.default_rng(N)
    a, b = (torch.from_numpy(rng.standard_normal((1, N, 64)).astype(np.float32)).cuda() for _ in range(2))
    gram = torch.from_numpy(rng.standard_normal((1, 64, 64)).astype(np.float32)).cuda()
    gram[0, 5, 5] = float("inf")
    got = ress.ress_block_drift_sq(a, b, gram, bq=128)
    assert bool((got == float("inf")).all()), got
