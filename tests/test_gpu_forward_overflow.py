"""Rasterizer.forward reads the pair count while the forward runs: a call
whose pairs do not fit grows the buffers and gives what a call on buffers that
were large enough gives (bit for bit), also on a stream of its own."""
import pytest
import torch

from paper_2601_19489_amd import scenes
from paper_2601_19489_amd.rasterizer import Rasterizer, params_to_device

pytestmark = pytest.mark.gpu

@pytest.mark.parametrize('deferred', [False, True])
@pytest.mark.parametrize('side_stream', [False, True])
def test_overflow_is_run_again(deferred, side_stream):
    d = scenes.surface_cloud(6000, seed=5, sh_degree=1, width=200, height=136)
    p = params_to_device(d)
    big = Rasterizer(6000, d['camera'], 1, capacity=1 << 20, deferred=deferred)
    big.forward(p)
    torch.cuda.synchronize()
    R = Rasterizer(6000, d['camera'], 1, capacity=1, deferred=deferred)
    st = torch.cuda.Stream() if side_stream else torch.cuda.current_stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        for _ in range(2):            # the first call grows the buffers, the second fits
            g = R.generation
            image, depth = R.forward(p)
            assert R.generation == g + 3
            assert R.pairs == big.pairs and R.capacity > R.pairs > 1000
            for got, want in ((image, big.image), (depth, big.depth),
                              (R.T_final, big.T_final), (R.n_contrib, big.n_contrib)):
                assert torch.equal(got, want)
        R.forward(p, check_overflow=False)
        assert R.pairs is None and torch.equal(R.image, big.image)
    st.synchronize()
