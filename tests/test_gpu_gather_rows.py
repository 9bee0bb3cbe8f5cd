"""The re-layout of a per-surfel field equals the copy by its map: row lengths around the copy units, an unaligned
field, few and many slots, an output shorter than the map."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# channels 4, 48 copy whole float4 rows (unless unaligned), 300 and 1,030 are longer than a workgroup's step
@pytest.mark.parametrize("n,short", [(1, 0), (255, 3), (4097, 0), (262_200, 1)])
@pytest.mark.parametrize("channels", [1, 3, 4, 5, 27, 48, 300, 1030])
def test_gather_equals_indexing(cuda, n, short, channels):
    import torch
    from paper_2411_00771_amd import raster
    if n > 5000 and channels > 48:
        n = 20_011
    rng = np.random.default_rng(n + channels)
    keep = np.flatnonzero(rng.random(n) < 0.9) if n > 1 else np.arange(n)
    new = np.sort(rng.integers(0, n, n // 5 + 1))
    src = np.concatenate([keep * 4, new * 4 + rng.integers(1, 4, len(new))])
    n_out = max(len(src) - short, 1)

    class Plan:
        counts = torch.tensor([0, 0, 0, 0, len(src)], dtype=torch.int64, device=cuda)

    smap = torch.from_numpy(src.astype(np.int32)).to(cuda)
    ids, kind = torch.from_numpy(src[:n_out] >> 2).to(cuda), torch.from_numpy(src[:n_out] & 3).to(cuda)
    for off in (0, 1):  # one float past an aligned start
        base = torch.randn(n * channels + 1, device=cuda)
        flat = base[off:off + n * channels]
        for zero_new in (False, True):
            live = (kind == 0) if zero_new else torch.ones_like(kind, dtype=torch.bool)
            g = raster.densify_gather(flat.view(n, channels), smap, Plan, n_out, blocked=True, zero_new=zero_new)
            assert torch.equal(g, flat.view(n, channels)[ids] * live[:, None]), (off, zero_new, "rows")
            g = raster.densify_gather(flat.view(channels, n), smap, Plan, n_out, zero_new=zero_new)
            assert torch.equal(g, flat.view(channels, n)[:, ids] * live), (off, zero_new, "planar")
