"""Both sides of the sizes from which a first pass no longer leaves its data in the cache for the second: one more
layer of a single element takes the vector across, and nothing may change in the layer before it."""
import pytest
import torch

from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu


def _first_layer(n, more, N, call, off):
    """Outputs of one step on the layer of n - off elements behind one of `off`, with or without the last layer."""
    sizes = ([off] if off else []) + [n - off] + ([1] if more else [])
    seg = [0]
    for k in sizes:
        seg.append(seg[-1] + k)
    P, at, gen = seg[-1], len(sizes) - 1 - int(more), torch.Generator(device="cuda")
    gen.manual_seed(n)

    def normal(std):
        t = torch.zeros(P, device="cuda")
        t[:n].normal_(0.0, std, generator=gen)
        return t

    q = QAdam(configs()[0], seg, N)
    g, e = [normal(1e-2) for _ in range(N)], [normal(1e-3) for _ in range(N)]
    want = [(a[off:n] + b[off:n]).abs().max() for a, b in zip(g, e)] if call != "w" else None
    codes = [torch.zeros(q.grad_code_bytes() // 4, dtype=torch.int32, device="cuda") for _ in range(N)]
    scales = [torch.zeros(len(sizes), device="cuda") for _ in range(N)]
    x, werr, wcodes = normal(0.02), torch.zeros(P, device="cuda"), torch.zeros(P, dtype=torch.int8, device="cuda")
    m = [torch.zeros(P, device="cuda") for _ in range(N if call == "w" else 1)]
    v = [torch.zeros(P, device="cuda") for _ in range(N if call == "w" else 1)]
    if call == "w":
        q.step_fused_w(1, 1e-3, 0.999, g, m, v, e, codes, scales, x, werr, wcodes)
    else:
        q.step_fused(1, 1e-3, 0.999, g, e, codes, scales, x, m[0], v[0], werr, wcodes)
    scales = [s[at].clone() for s in scales]
    if want:
        assert all(torch.equal(s, w) for s, w in zip(scales, want))
    assert q.get_status() == 0
    q.close()
    return [x[off:n].clone(), werr[off:n].clone(), wcodes[off:n].clone()] + [b[off:n].clone() for b in e + m + v] + scales


@pytest.mark.parametrize("call,N,limit", [("s", 1, (192 << 20) // 8), ("s", 4, (768 << 20) // 32), ("w", 2, (512 << 20) // 8)])
@pytest.mark.parametrize("off", [0, 1001])
def test_one_element_across_the_limit(call, N, limit, off):
    below = _first_layer(limit, False, N, call, off)
    beyond = _first_layer(limit, True, N, call, off)
    assert all(torch.equal(a, b) for a, b in zip(below, beyond))
