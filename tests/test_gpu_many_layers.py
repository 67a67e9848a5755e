"""GPU parity on lists of very many layers, where the scales are found a workgroup per 16 layers and the launches come
near their largest size.  Bit for bit against the oracle, which takes such a list in one call."""
import numpy as np
import pytest
import torch

from oracle import qadam_oracle as oracle
from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu


def _same(dev, host):
    return np.array_equal(dev.cpu().numpy().view(np.uint8), np.ascontiguousarray(host).view(np.uint8))


def _step(sizes, N, call, seed, status=0, bad=(), **cfgkw):
    """One step from a state that is nowhere zero; every output compared with the oracle's.  bad: elements of the first
    worker's gradient that are infinite."""
    gcfg, ocfg = configs(**cfgkw)
    seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    P, L, rng = int(seg[-1]), len(sizes), np.random.default_rng(seed)
    f32 = lambda s: rng.standard_normal(P, dtype=np.float32) * np.float32(s)  # noqa: E731
    dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
    hg, he = [f32(1e-2) for _ in range(N)], [f32(1e-3) for _ in range(N)]
    hg[0][list(bad)] = np.inf
    hx, hw = f32(0.02), f32(1e-3)
    nm = N if call[0] == "w" else 1
    hm, hv = [f32(1e-3) for _ in range(nm)], [f32(1e-3) ** 2 for _ in range(nm)]
    g, e, m, v = ([dev(a) for a in b] for b in (hg, he, hm, hv))
    x, werr = dev(hx), dev(hw)
    wcodes = torch.full((P,), 77, dtype=torch.int8 if gcfg.k_x <= 6 else torch.int16, device="cuda")
    q = QAdam(gcfg, seg.tolist(), N)
    codes = [torch.full((q.grad_code_bytes() // 4,), -1, dtype=torch.int32, device="cuda") for _ in range(N)]
    scales = [torch.full((L,), -1.0, device="cuda") for _ in range(N)]
    if call == "fused":
        q.step_fused(1, 1e-3, 0.999, g, e, codes, scales, x, m[0], v[0], werr, wcodes)
    elif call == "calls":
        for i in range(N):
            q.worker_quantize(i, 1, g[i], e[i], codes[i], scales[i])
        q.server_step(1, 1e-3, 0.999, codes, scales, x, m[0], v[0])
        q.weight_quantize(1, x, werr, wcodes)
    elif call == "w":
        q.step_fused_w(1, 1e-3, 0.999, g, m, v, e, codes, scales, x, werr, wcodes)
    elif call == "w_calls":
        for i in range(N):
            q.worker_step_w(i, 1, 1e-3, 0.999, g[i], m[i], v[i], e[i], codes[i], scales[i])
        q.server_apply_w(1, codes, scales, x)
        q.weight_quantize(1, x, werr, wcodes)
    if call[0] == "w":
        out = oracle.step_w(ocfg, seg, 1, 1e-3, 0.999, hg, he, hm, hv, hx, hw, want_tie=False)
    else:
        out = oracle.step_s(ocfg, seg, 1, 1e-3, 0.999, hg, he, hx, hm[0], hv[0], hw, want_tie=False)
    assert q.get_status() == status
    for i in range(N):
        assert _same(scales[i], out["scales"][i]) and _same(codes[i], out["words"][i]) and _same(e[i], he[i]), (call, i)
    assert all(_same(a, b) for a, b in zip(m + v + [x, werr, wcodes], hm + hv + [hx, hw, out["wcodes"]])), call
    q.close()


T = 4096


@pytest.mark.parametrize("call", ["fused", "calls", "w"])
@pytest.mark.parametrize("N", [1, 3])
def test_layers_each_side_of_a_wavefronts_turn(call, N):
    """Layers of 511 to 513 maxima (one per tile, four in variant W) among short and empty ones; 1025 layers or more, so
    that a workgroup takes 16 layers also with one worker, the last one fewer."""
    long = [T * 512 - 3, T * 512 + 1, T * 128, T * 128 + 5] if N == 1 else [T * 512 + 1, T * 128, T * 128 + 1]
    sizes = [1, 33, 0, 1000, 5] * 100 + long + [7, 255, 1025, 0, 3] * 105
    assert len(sizes) > 1024 and len(sizes) % 16
    _step(sizes, N, call, seed=11 + N)


@pytest.mark.parametrize("call", ["fused", "calls", "w"])
def test_more_layers_than_workgroups_of_1024_threads_fit(call):
    """2^22 + 5 layers: a workgroup of 1024 threads for each would be a launch of 2^32 work-items."""
    _step([1] * ((1 << 22) + 4) + [3 * T + 1], 1, call, seed=3)


@pytest.mark.parametrize("call", ["calls", "w_calls"])
def test_whole_tiles_where_the_quantizers_pieces_are_longer_than_a_turn(call):
    """2^23 tiles: the worker quantizer's launch then holds four pieces per tile, each two turns of a wavefront.  Most
    tiles are layers of one element; two layers have whole tiles, one of them off the 16-byte grid."""
    _step([3 * T + 700, 1025] + [1] * (1 << 23) + [2 * T + 2600], 1, call, seed=4)


@pytest.mark.parametrize("call", ["fused", "calls", "w", "w_calls"])
@pytest.mark.parametrize("sizes,N", [
    ([600] * 800 + [3], 2),                                     # three pieces of 256, two of 512, one of 1024
    ([1023, 513, 1025, 7] * 300, 3),                            # five pieces of 256: one more than a quarter of a tile
    ([T, 64, 64, 64, 64, 64, 64, 64, 65] * 1100, 1),            # sparse: longer pieces, on and off the 16-byte grid
    ([T * 2000 + 5] + [100] * 9000, 1),                         # one long layer and many short ones
])
def test_pieces_of_short_and_mixed_layers(call, sizes, N):
    _step(sizes, N, call, seed=len(sizes))
