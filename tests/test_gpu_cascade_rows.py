"""GPU: the standalone cascade over more rows than it has places (64 in flight
when a row takes several shards): a place's next row must find the barrier
state and the top-p histograms as the first one did."""
import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,top_p,second", [(4100, 0.9, True), (4100, 1.0, True), (20000, 0.7, True), (65536, 0.95, False)])
def test_long_row_lists_equal_short_ones(V, top_p, second):
    import torch
    from paper_2609_17184_amd.binding import cascade
    rows = 150
    g = torch.Generator().manual_seed(3)
    zR = 2.0 * torch.randn(rows, V, generator=g)
    z1 = (zR + 0.8 * torch.randn(rows, V, generator=g)).cuda()
    z2 = (zR + 0.4 * torch.randn(rows, V, generator=g)).cuda() if second else None
    zR = zR.cuda()
    keys = torch.stack([torch.arange(rows), torch.arange(rows) * 7 + 1], 1).int().cuda()
    log(f"[cascade] {rows} rows of {V}, top-p {top_p}")
    whole = [t.cpu().numpy() for t in cascade(z1, z2, zR, keys, 1.0, top_p)]
    for a, b in ((0, 50), (50, 100), (100, 150)):
        part = cascade(z1[a:b], z2[a:b] if second else None, zR[a:b], keys[a:b].contiguous(), 1.0, top_p)
        for x, y in zip(whole, part):
            assert np.array_equal(x[a:b], y.cpu().numpy()), (V, a)
    assert set(np.unique(whole[0][:, 1])) >= {0, 1}              # both accepted and resampled rows among them
