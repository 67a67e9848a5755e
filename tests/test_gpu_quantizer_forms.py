"""GPU parity of the gradient quantizer where its two forms meet: scales on both sides of the range in which the quotient is a
product and sums take one rounding (2^-100 .. 2^100), zeros of both signs, subnormals, levels and midpoints, for every grid.
Equal bit for bit: both sides execute the same binary32 operations in the same order, but for sums that take one rounding with an
exact product, which is the same.  A residual of zero is +0 on the device, where a zero message has the sign of p; the oracle's message is
+0, and its residual of p = -0 is -0."""
import numpy as np
import pytest
import torch

from oracle import qadam_oracle as oracle
from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu

UP, DOWN = np.float32(2.0 ** 100), np.float32(2.0 ** -100)
SCALES = [1.0, 0.37, UP, np.nextafter(UP, np.float32(np.inf)), DOWN, np.nextafter(DOWN, np.float32(0)), 0.0, 1e-44, 3e-39, 2.0 ** 127]


def _bits(a):
    return a.view(np.uint32)


def _plus_zero(e):
    return e + np.float32(0.0)          # -0 + 0 is +0; nothing else changes


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
        assert np.array_equal(_bits(e.cpu().numpy()), _bits(_plus_zero(he))), fused
        assert np.array_equal(codes.cpu().numpy().view(np.uint32), want["words"]), fused
    q.close()


@pytest.mark.parametrize("k_g", range(7))
@pytest.mark.parametrize("n", [256, 1000, 4099])
def test_sums_over_workers_give_the_oracles_moments_and_weights(k_g, n):
    """The workers' scales of a layer differ, so that both forms add to one sum; where they are close to each other its additions round."""
    workers, list_of = 4, SCALES[:-1] + [2.0 ** 124]        # sums over workers stay finite
    gcfg, ocfg = configs(k_g=k_g)
    rng = np.random.default_rng(10 * k_g + n)
    parts = [[_layer(list_of[(l + 3 * i) % len(list_of)] if i % 2 else s * (1 + i / 10), k_g, n, rng) for l, s in enumerate(list_of)]
             for i in range(workers)]
    hg, he = ([np.concatenate([p[k] for p in parts[i]]) for i in range(workers)] for k in (0, 1))
    seg = (np.arange(len(list_of) + 1) * n).astype(np.int64)
    P = int(seg[-1])
    hx = (rng.standard_normal(P) * 0.02).astype(np.float32)
    hm, hv, hw = (np.zeros(P, np.float32) for _ in range(3))
    dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
    q = QAdam(gcfg, seg.tolist(), workers)
    g, e, x, m, v, w = [dev(a) for a in hg], [dev(a) for a in he], dev(hx), dev(hm), dev(hv), dev(hw)
    scales = [torch.zeros(len(list_of), device="cuda") for _ in range(workers)]
    codes = [torch.full((q.grad_code_bytes() // 4,), -1, dtype=torch.int32, device="cuda") for _ in range(workers)]
    wcodes = torch.zeros(P, dtype=torch.int8, device="cuda")
    for t in (1, 2):
        want = oracle.step_s(ocfg, seg, t, 1e-3, 0.999, hg, he, hx, hm, hv, hw)
        q.step_fused(t, 1e-3, 0.999, g, e, codes, scales, x, m, v, w, wcodes)
        for i in range(workers):
            assert np.array_equal(_bits(scales[i].cpu().numpy()), _bits(want["scales"][i])), (t, i)
            assert np.array_equal(codes[i].cpu().numpy().view(np.uint32), want["words"][i]), (t, i)
        for name, got, host in [("e%d" % i, e[i], _plus_zero(he[i])) for i in range(workers)] + [("x", x, hx), ("m", m, hm), ("v", v, hv), ("e^x", w, hw)]:
            assert np.array_equal(_bits(got.cpu().numpy()), _bits(host)), (t, name)
        assert np.array_equal(wcodes.cpu().numpy(), want["wcodes"]), t
    q.close()
