"""The depth sort around the sizes where its passes change: one tile of 2048
keys, one group of 32 tiles, and 2^22 keys (above which a pass scans its
histogram in launches of its own). One 16 x 16 tile that every splat covers:
its list is the depth order, ties by index (exact)."""
import numpy as np
import pytest
import torch

from paper_2601_19489_amd import _lib, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n', [1, 2, 255, 2047, 2048, 2049, 65535, 65536, 65537, 300_001,
                               1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize('ties', [False, True])
def test_one_tile_list_is_the_stable_depth_order(n, ties):
    cam = scenes.look_at_camera((0, 0, -4), (0, 0, 0), 16, 16, tile=16)
    ccam = _lib.camera(cam, 16)
    g = torch.Generator(device='cuda').manual_seed(n)
    if ties:  # few distinct keys, over all four digits
        some = torch.tensor([0x3F800000, 0x3F800001, 0x40490FDB, 0x40490EDB, 0x7F7FFFFF, 1],
                            dtype=torch.int32, device='cuda')
        keys = some[torch.randint(len(some), (n,), generator=g, device='cuda')]
    else:
        keys = torch.randint(0, 0x7F800000, (n,), generator=g, device='cuda', dtype=torch.int32)
    rec = torch.zeros((n, _lib.SPLAT_FLOATS), device='cuda')
    rec[:, 0:2] = 8.0
    rec[:, 2] = rec[:, 4] = 1e-3
    rec[:, 5] = 2.0 * float(np.log(255.0 * 0.5))
    rec[:, 6] = 0.5
    rec.view(torch.int32)[:, 11] = 1 << 16            # columns 0 .. 0
    counts = torch.ones(n, dtype=torch.int32, device='cuda')
    ws = torch.empty(_lib.gs_bin_sort_workspace(n, n, ccam), dtype=torch.uint8, device='cuda')
    ws.fill_(0xA5)                                    # nothing is taken as zero
    vals = torch.full((n,), -1, dtype=torch.int32, device='cuda')
    ranges = torch.empty(2, dtype=torch.int32, device='cuda')
    pairs = torch.zeros(1, dtype=torch.int32, device='cuda')
    for _ in range(2):                                # and again on the used workspace
        _lib.gs_bin_sort(rec, keys, counts, n, ccam, ws, n, vals, ranges, None, pairs)
    torch.cuda.synchronize()
    assert pairs.item() == n and ranges.tolist() == [0, n]
    want = np.argsort(keys.cpu().numpy().view(np.uint32), kind='stable')
    np.testing.assert_array_equal(vals.cpu().numpy(), want)
