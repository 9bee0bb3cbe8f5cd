"""Codeword assignment and update at the edges of their tiles: dimensions padded to the matrix steps, chunks of 128
codewords, whole rounds of workgroups and the split rest."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,K", [(1, 1), (3, 15), (4, 129), (9, 16), (12, 256), (25, 127), (27, 300), (28, 128),
                                 (45, 257), (48, 130)])
# a row of a tile, a split workgroup short and full, 128 whole ones and one more row, a whole round and a rest
@pytest.mark.parametrize("m", [1, 31, 33, 4097, 16_385, 131_109])
def test_assign_is_the_nearest(cuda, D, K, m):
    import torch
    from paper_2411_00771_amd import storage
    g = torch.Generator(device=cuda).manual_seed(m + D)
    n = m + 77
    x = torch.randn(n, D, device=cuda, generator=g)
    rows = torch.randperm(n, device=cuda, generator=g)[:m].sort().values.to(torch.int32)
    cb = torch.randn(K, D, device=cuda, generator=g)
    if K > 2:
        cb[K - 1] = cb[1]  # of equal codewords the first is taken
    code = storage.vq_assign(x, D, rows, cb).to(torch.int64) & 0xffff
    q, c = x[rows.long()].double(), cb.double()
    score = (c * c).sum(1) - 2 * q @ c.T
    took = score.gather(1, code[:, None])[:, 0]
    # products and sums of FP32: D + 3 roundings of at most |c|^2 + 2 |x| |c| on either of the two scores
    size = (c * c).sum(1).max() + 2 * q.norm(dim=1) * c.norm(dim=1).max()
    assert bool((took <= score.min(1).values + 2 * (D + 3) * 2.0 ** -24 * size).all())
    if K > 2:
        assert not bool((code == K - 1).any())


@pytest.mark.parametrize("D,K", [(1, 3), (12, 256), (27, 1000), (48, 70)])
@pytest.mark.parametrize("m", [1, 63, 65, 30_011])
def test_update_is_the_mean(cuda, D, K, m):
    import torch
    from paper_2411_00771_amd import storage
    rng = np.random.default_rng(m + D)
    x = torch.from_numpy(rng.standard_normal((m, D)).astype(np.float32)).to(cuda)
    rows = torch.arange(m, device=cuda, dtype=torch.int32)
    raw = np.minimum(rng.geometric(0.01, m) - 1, K + 1)  # a popular codeword, and some past the codebook
    raw[::7] = rng.integers(0, K, len(raw[::7]))
    code = torch.from_numpy(raw.astype(np.uint16).view(np.int16)).to(cuda)
    cb = torch.full((K, D), 7.0, device=cuda)
    counts = storage.vq_update(x, D, rows, code, cb).cpu().numpy()
    want = np.full((K, D), 7.0)
    for k in range(K):
        sel = raw == k
        if sel.any():
            want[k] = x.cpu().numpy()[sel].astype(np.float64).mean(0)
    assert np.array_equal(counts, np.bincount(raw[raw < K], minlength=K))
    # FP64 sums in another order, rounded once: one unit in the last place, and the sums' cancellation
    assert np.allclose(cb.cpu().numpy(), want, rtol=2.0 ** -23, atol=1e-12)
