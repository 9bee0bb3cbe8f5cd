"""The view sums and counters of the densification statistics at the edges of their blocks (1,024 surfels a sum) and of
the short form (up to 32,768 surfels)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,V,density", [(1, 1, 1.0), (63, 2, 0.5), (1023, 1, 0.9), (1024, 3, 0.1),
                                         (1025, 2, 1.0), (100, 64, 0.5), (32_768, 3, 0.2), (32_769, 2, 0.2),
                                         (1_050_000, 2, 0.04)])
def test_block_edges_match_oracle(cuda, n, V, density):
    import torch
    from paper_2411_00771_amd import raster
    rng = np.random.default_rng(n)
    ls = rng.normal(-4, 1, (2, n)).astype(np.float32)
    z = lambda *s: torch.zeros(s, device=cuda)
    params = raster.Params(z(3, n), torch.from_numpy(ls).to(cuda), z(4, n), z(n), z(n, 1, 3), 0)
    eng = raster.Engine(n, 16, 16, V, capacity=1 << 10)
    flags = ((rng.random((V, n)) < density) * 1).astype(np.uint8)
    flags[:, -1] = 1 | 32  # the ragged end counts
    flags[:, :-1] |= ((rng.random((V, n - 1)) < 0.1) * 32).astype(np.uint8)
    radius = rng.uniform(0, 20, (V, n)).astype(np.float32)
    gt = rng.normal(0, 1e-5, (V, 2, n)).astype(np.float32)
    gs = rng.normal(0, 3e-6, (V, 2, n)).astype(np.float32)
    eng.flags[:V * n].copy_(torch.from_numpy(flags.reshape(-1)))
    eng.radius[:V * n].copy_(torch.from_numpy(radius.reshape(-1)))
    g = raster.Grads(params, V)
    g.g_view_total.copy_(torch.from_numpy(gt))
    g.g_view_ssim.copy_(torch.from_numpy(gs))
    st = raster.DensifyState(n, V)
    eng.densify(params, g, st, omega=0.9, eta_min=0.05, grad_threshold=2e-6)
    torch.cuda.synchronize()
    ost = oracle.new_densify_state(n)
    total = np.zeros(6, np.int64)
    for v in range(V):
        vis = (flags[v] & 1) > 0
        lp = (flags[v] & 32) > 0
        r = oracle.densify_stats(gt[v].T, gs[v].T, vis, radius[v], ls, ost, 0.9, 0.05, 2e-6, lowpass=lp)
        # the sums are FP64 on both sides; the scale is stored in FP32
        assert abs(st.scale[v].item() / r["scale"] - 1) <= 2.0 ** -23, v
        total[[0, 4]] += vis.sum(), (vis & lp).sum()
    # at most V + 1 roundings of terms of one sign, the FP32 norm's two and the scale's
    bound = (V + 5) * 2.0 ** -23
    assert np.allclose(st.accum_dgd.cpu().numpy(), ost["accum_dgd"], rtol=bound, atol=1e-30)
    assert np.array_equal(st.denom.cpu().numpy(), ost["denom"])
    assert np.array_equal(st.max_radius.cpu().numpy(), ost["max_radius"].astype(np.float32))
    m = st.mask.cpu().numpy()
    c = st.counters.cpu().numpy()
    total[[1, 2, 3, 5]] = (m & 1).sum(), ((m >> 1) & 1).sum(), ((m & 3) == 3).sum(), ((m >> 2) & 1).sum()
    assert np.array_equal(c[:6], total)
