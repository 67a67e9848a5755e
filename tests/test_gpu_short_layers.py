"""GPU parity of layers that one workgroup takes from the gradient to the codes: ends of each size of workgroup, both sides of
the rule that sets such layers apart, and lists where they stand beside longer and empty ones."""
import numpy as np
import pytest
import torch

from paper_2004_14180_amd import QAdam
from parity_util import DeviceState, configs
from test_gpu_many_layers import _step
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

CALLS = ["fused", "calls", "w", "w_calls"]
ENDS = [1, 3, 33, 255, 256, 257, 0, 511, 1000, 1023, 1024, 64]          # one wavefront, four
TILE = [1025, 2047, 4093, 4095, 4096]                                   # four wavefronts with four quads per lane
SETTINGS = [dict(), dict(k_g=0, k_x=14), dict(k_g=6, rounding=1), dict(eps=0.0, adam_flavor=1)]


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("cfgkw", SETTINGS)
@pytest.mark.parametrize("N", [1, 3])
def test_ends_of_each_size(call, cfgkw, N):
    """Every layer on and off the 16-byte grid; all three sizes in launches of their own, or the fewer with the next."""
    _step(ENDS * 3, N, call, seed=1, **cfgkw)
    _step(ENDS * 60 + TILE * 52, N, call, seed=2, **cfgkw)
    _step(ENDS[:3] * 20 + TILE * 60, N, call, seed=3, **cfgkw)


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("sizes,N", [
    ([1000] * 319 + [1025], 1), ([1000] * 318 + [1025], 1),             # with layers of more than 1024: from 320 on
    ([100, 700] * 20, 8), ([100, 700] * 20, 9), ([100] * 320, 9),       # without: from eight workers on likewise
    ([9000] + [65] * 2047, 1), ([9000] + [65] * 2048, 1),               # beside longer layers: from 2048 on
    ([5000, 100, 1100, 0] * 1100 + [4097, 300], 5),
])
def test_each_side_of_the_rule(call, sizes, N):
    _step(sizes, N, call, seed=len(sizes) + N)


@pytest.mark.parametrize("call", ["calls", "w_calls"])
@pytest.mark.parametrize("sizes,N", [(([4096] + [64] * 16) * 500, 3), (([9001] + [64] * 20 + [0, 700]) * 400, 4)])
def test_server_by_section(call, sizes, N):
    """Lists whose server takes each size of short layers, and the longer ones, in launches of their own."""
    _step(sizes, N, call, seed=N)


@pytest.mark.parametrize("call", ["fused", "calls"])
def test_infinite_gradients(call):
    """In a layer of each size: its scale is infinite, its codes are zero, the status word says so."""
    _step([200] * 300 + [1000] * 300 + [3000] * 300, 2, call, seed=4, status=1,
          bad=(200 * 7 + 5, 200 * 300 + 1000 * 8 + 999, 1200 * 300 + 3000 * 299 + 2500))


@pytest.mark.parametrize("trust", [2, 3])
@pytest.mark.parametrize("cfgkw", [dict(), dict(weight_ef=0), dict(k_g=1, rounding=1, seed=2)])
def test_beside_a_filtered_scale_pass(trust, cfgkw):
    rep, st = _custom([70000, 40] + [500, 4096, 1] * 700 + [0, 20001], 3, 3, seed=6, cfgkw=cfgkw, trust=trust)
    assert rep.ok() and st == 0, rep.line()


def test_replayed_from_a_graph():
    seg = np.concatenate([[0], np.cumsum([300] * 1500 + [30000] + [2000] * 600)])
    N = 3
    qa, qb = QAdam(configs()[0], seg, N), QAdam(configs()[0], seg, N)
    gen = torch.Generator().manual_seed(5)
    x0 = torch.randn(int(seg[-1]), generator=gen) * 0.02
    a, b = DeviceState(qa, x0), DeviceState(qb, x0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.step_fused(1, 1e-3, 0.999)
    for t in range(1, 5):
        for i in range(N):
            g = torch.randn(x0.numel(), generator=gen) * 0.01
            a.grads[i].copy_(g); b.grads[i].copy_(g)
        graph.replay()
        b.step_fused(t, 1e-3, 0.999)
        torch.cuda.synchronize()
        assert all(torch.equal(getattr(a, k), getattr(b, k)) for k in ("x", "m", "v", "werr", "wcodes")), t
        assert all(torch.equal(u, w) for k in ("errs", "codes", "scales") for u, w in zip(getattr(a, k), getattr(b, k))), t
        assert (a.x * 2).sum().isfinite()
    qa.close(); qb.close()
