"""The trimming bound for one to more workgroups than histogram copies, and over a captured graph's replays (the passes
leave the copies cleared)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2048, 2049, 3 * 2048, 8 * 2048, 9 * 2048 + 1, 1_000_003])
def test_bound_is_the_sorted_element(cuda, n):
    import torch
    from paper_2411_00771_amd import raster
    rng = np.random.default_rng(n)
    c = np.where(rng.random(n) < 0.3, 0, rng.lognormal(-3, 4, n)).astype(np.float32)
    c[rng.integers(0, n, max(n // 50, 1))] = np.float32(0.25)
    for ratio in (0.0, 0.03125, 0.5, 0.9375):  # exact in float32, as the library takes it
        bound, mask, removed = raster.trim_mask(torch.from_numpy(c).to(cuda), ratio)
        b_ref, m_ref = oracle.trim_threshold(c, ratio)
        assert np.float32(bound.item()) == np.float32(b_ref), ratio
        assert np.array_equal(mask.cpu().numpy().astype(bool), m_ref)
        assert removed.item() == int(m_ref.sum())


def test_replays(cuda):
    import torch
    from paper_2411_00771_amd import raster
    c = torch.rand(50_000, device=cuda)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        raster.trim_mask(c, 0.1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bound, mask, removed = raster.trim_mask(c, 0.1)
    for k in range(4):
        c.copy_(torch.rand(50_000, device=cuda))
        graph.replay()
        torch.cuda.synchronize()
        b_ref, m_ref = oracle.trim_threshold(c.cpu().numpy(), 0.1)
        assert np.float32(bound.item()) == np.float32(b_ref), k
        assert np.array_equal(mask.cpu().numpy().astype(bool), m_ref), k
