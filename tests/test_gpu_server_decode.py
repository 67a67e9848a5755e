"""GPU parity of the server's decoding where its two forms meet: scales on both sides of the range that the form for four
elements at once is used in (2^-100 .. 2^100), mixed among the workers of one layer, for every width of a code and numbers
of workers around the loop's unrolling.  Bit for bit: both sides execute the same binary32 operations in the same order."""
import numpy as np
import pytest
import torch

from oracle import qadam_oracle as oracle
from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu

SIZES = [1, 31, 33, 255, 256, 257, 4097, 1000, 5]
UP, DOWN = np.float32(2.0 ** 100), np.float32(2.0 ** -100)
SCALES = np.array([1.0, 0.37, UP, np.nextafter(UP, np.float32(np.inf)), DOWN, np.nextafter(DOWN, np.float32(0)), 0.0, 1e-44,
                   3e-39], np.float32)


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 9, 16, 32])
@pytest.mark.parametrize("k_g", [0, 1, 2, 6])
def test_server_step_for_scales_of_every_size(N, k_g):
    gcfg, ocfg = configs(k_g=k_g)
    seg = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    P, L, rng = int(seg[-1]), len(SIZES), np.random.default_rng(100 * k_g + N)
    f32 = lambda s: rng.standard_normal(P).astype(np.float32) * np.float32(s)  # noqa: E731
    words = [oracle.worker_quantize(ocfg, seg, i, 1, f32(1.0), f32(0.1))["words"] for i in range(N)]
    for case in range(3):
        # all workers of a layer ordinary / each with another of the values / one worker out of the range
        scales = [np.full(L, 0.5 + 0.01 * i, np.float32) for i in range(N)]
        for i in range(N):
            if case == 1 or (case == 2 and i == N - 1):
                scales[i][:] = np.roll(SCALES, i + case)[:L]
        hx, hm, hv = f32(0.02), f32(1e-3), f32(1e-3) ** 2
        dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
        x, m, v = dev(hx), dev(hm), dev(hv)
        q = QAdam(gcfg, seg.tolist(), N)
        q.server_step(1, 1e-3, 0.999, [dev(w.view(np.int32)) for w in words], [dev(s) for s in scales], x, m, v)
        oracle.server_step(ocfg, seg, 1, 1e-3, 0.999, words, scales, hx, hm, hv)
        for a, b in ((x, hx), (m, hm), (v, hv)):
            assert np.array_equal(a.cpu().numpy().view(np.int32), b.view(np.int32)), case
        q.close()
