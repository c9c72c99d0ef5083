"""A pruned Gaussian has no output entry, and its rows are not read: an event
that prunes almost everything costs a fraction of one that copies everything
(1M Gaussians of 59 values; the copy reads and writes 472 MB, the pruning 8 MB.
Reading the rows of what is pruned as well takes 0.38 of the copy's time,
leaving them out 0.10; the bar is 0.3)."""
import pytest
import torch

from paper_2601_19489_amd import _lib

pytestmark = pytest.mark.gpu

NAMES = ('means', 'log_scales', 'quats', 'opacity_logits', 'sh')
N, DEG = 1_000_000, 3


def _time(p, eps, kinds, moments):
    n_of = torch.tensor([1, 2, 2, 0], device='cuda')[kinds.long()]
    n_out = int(n_of.sum())
    ws = torch.zeros(_lib.gs_densify_workspace(N), dtype=torch.uint8, device='cuda')
    ws.view(torch.int32)[:N] = (torch.cumsum(n_of, 0) - n_of).to(torch.int32)   # offsets, kinds
    ws.view(torch.int32)[N:2 * N] = kinds
    out = {k: torch.empty(v.shape[:-1] + (n_out,), device='cuda') for k, v in p.items()}
    g, o = (_lib.gaussians(*(d[k] for k in NAMES)) for d in (p, out))
    best = float('inf')
    for _ in range(20):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(5):
            _lib.gs_densify_apply(g, N, DEG, None if moments else eps, ws, n_out, moments, o)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 5)
    return best, out


@pytest.mark.parametrize('moments', [0, 1])
def test_pruned_rows_are_not_read(moments):
    g = torch.Generator(device='cuda').manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g, device='cuda')
    p = dict(means=rnd(3, N), log_scales=rnd(3, N) - 3, quats=rnd(4, N), opacity_logits=rnd(N),
             sh=rnd((DEG + 1) ** 2, 3, N))
    eps = rnd(2, 3, N)
    copy = torch.zeros(N, dtype=torch.int32, device='cuda')
    prune = torch.full_like(copy, 3)
    prune[777_777] = 0
    t_copy, same = _time(p, eps, copy, moments)
    t_prune, kept = _time(p, eps, prune, moments)
    for k, v in p.items():
        assert torch.equal(same[k], v), k
        assert torch.equal(kept[k][..., 0], v[..., 777_777]), k
    assert t_prune < 0.3 * t_copy, (t_prune, t_copy)
