"""GPU parity of the gradient quantizer where its two forms meet: scales on both sides of the range in which the quotient is a
product and sums take one rounding (2^-100 .. 2^100), zeros of both signs, subnormals, levels and midpoints, for every grid.
Equal, but for the sign of a zero: both sides execute the same binary32 operations in
the same order."""
import numpy as np
import pytest
import torch

from oracle import qadam_oracle as oracle
from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu

UP, DOWN = np.float32(2.0 ** 100), np.float32(2.0 ** -100)
SCALES = [1.0, 0.37, UP, np.nextafter(UP, np.float32(np.inf)), DOWN, np.nextafter(DOWN, np.float32(0)), 0.0, 1e-44, 3e-39, 2.0 ** 127]


def _layer(s, k_g, n, rng):
    """(g, e) of a layer with scale s."""
    s = np.float32(s)
    marks = [2.0 ** (-k_g - 1)] + [c * 2.0 ** -j for j in range(k_g + 1) for c in (0.75, 1.0)]
    g = (rng.uniform(-1, 1, n) * 2.0 ** rng.uniform(-12, 0, n)).astype(np.float32) * s
    for i, m in enumerate(marks):
        v = np.float32(np.float64(s) * m)
        g[2 + 4 * i:6 + 4 * i] = [v, -v, np.nextafter(v, np.float32(0)), -np.nextafter(v, np.float32(0))]
    g[-12:-4] = np.array([0.0, -0.0, 0.0, -0.0, 1e-45, -1e-45, 1e-39, -1e-39], np.float32)
    e = np.zeros(n, np.float32)
    e[-12:-4] = np.array([0.0, -0.0, -0.0, 0.0, 0.0, -0.0, -0.0, 0.0], np.float32)
    e[n // 2:n // 2 + 40] = -g[n // 2:n // 2 + 40]              # sums that cancel
    g = np.clip(g, -s, s)
    g[0] = s
    return g, e


@pytest.mark.parametrize("k_g", range(7))
@pytest.mark.parametrize("n", [256, 1000, 4099])
def test_every_form_gives_the_oracles_values(k_g, n):
    gcfg, ocfg = configs(k_g=k_g)
    rng = np.random.default_rng(10 * k_g + n)
    parts = [_layer(s, k_g, n, rng) for s in SCALES]
    hg, he = (np.concatenate([p[i] for p in parts]) for i in (0, 1))
    seg = (np.arange(len(SCALES) + 1) * n).astype(np.int64)
    want = oracle.worker_quantize(ocfg, seg, 0, 1, hg, he)
    dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
    he0 = np.concatenate([p[1] for p in parts])
    q = QAdam(gcfg, seg.tolist(), 1)
    for fused in (False, True):
        g, e, scales = dev(hg), dev(he0), torch.zeros(len(SCALES), device="cuda")
        codes = torch.full((q.grad_code_bytes() // 4,), -1, dtype=torch.int32, device="cuda")
        if fused:
            f = lambda: torch.zeros(hg.size, device="cuda")  # noqa: E731
            q.step_fused(1, 1e-3, 0.999, [g], [e], [codes], [scales], f(), f(), f(), f(), torch.zeros(hg.size, dtype=torch.int8, device="cuda"))
        else:
            q.worker_quantize(0, 1, g, e, codes, scales)
        assert np.array_equal(e.cpu().numpy(), he), fused
        assert np.array_equal(codes.cpu().numpy().view(np.uint32), want["words"]), fused
    q.close()
