"""GPU parity where the size of a vector decides how its scales are found: by the quantizing kernel itself on short
vectors, by a launch of their own on longer ones, and in the one workgroup that does a whole short segment.
Everything is compared bit for bit (the oracle executes the same binary32 operations in the same order)."""
import numpy as np
import pytest
import torch

from paper_2004_14180_amd import QAdam
from paper_2004_14180_amd.binding import quantize_segment_noalloc
from parity_util import configs
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

T = 4096


@pytest.mark.parametrize("N,tiles", [(1, 128), (8, 128), (8, 129), (4, 256), (4, 257), (1, 1024), (1, 1025)])
@pytest.mark.parametrize("fused", [True, False])
def test_each_side_of_the_fold(N, tiles, fused):
    # one long layer, one off the 16-byte grid, one of a single element
    sizes = [(tiles - 3) * T - 5, T + 2, 1]
    rep, st = _custom(sizes, N, 2, seed=tiles, fused=fused, trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("layers,tiles", [(32, 64), (33, 64), (31, 65), (1024, 2), (1025, 2)])
@pytest.mark.parametrize("fused", [True, False])
def test_one_worker_each_side_of_the_fold_of_short_layers(layers, tiles, fused):
    """Twice the tiles for one worker where no layer has more than 64 of them."""
    rep, st = _custom([tiles * T - 6] * layers, 1, 1, seed=layers + tiles, fused=fused)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("N,longest,others", [(1, 768, 0), (1, 769, 0), (1, 700, 324), (1, 700, 325), (2, 384, 0), (2, 385, 0),
                                              (2, 512, 0), (2, 513, 0), (4, 96, 160), (4, 97, 0), (10, 1, 101), (10, 1, 102),
                                              (11, 1, 50), (16, 64, 0), (16, 65, 0), (16, 1, 126)])
@pytest.mark.parametrize("fused", [True, False])
def test_each_side_of_the_longest_folded_layer(N, longest, others, fused):
    """The limits on the longest layer's tiles, on tiles times workers and on elements times workers."""
    sizes = [3] + [T - 1] * (others - 1) + [longest * T - 6] if others else [longest * T - 6]
    rep, st = _custom(sizes, N, 2, seed=longest + N, fused=fused, trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("N", [3, 5, 6])
@pytest.mark.parametrize("w", [False, True])
def test_folded_workers_beyond_whole_groups(N, w):
    """Two or five workers are folded together: the last group is not whole.  Layers of more than 64 maxima and of one, and the ends of
    layers, which are folded the same way."""
    sizes = [66 * T + 9, 1, 255, T, 700]
    if w:
        _worker_moments(N, 70, sizes)
    else:
        rep, st = _custom(sizes, N, 2, seed=N, trust=2)
        assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("N,tiles", [(2, 128), (8, 129), (4, 255), (4, 257)])
def test_worker_moments_each_side_of_the_fold(N, tiles):
    """Variant W leaves four maxima per tile: ends of a layer in each quarter of its last tile."""
    _worker_moments(N, tiles, [(tiles - 5) * T, 1000, T + 1025, 3, 2049])


@pytest.mark.parametrize("N,tiles", [(1, 192), (1, 193), (2, 96), (2, 97), (4, 24), (4, 25), (1, 256), (1, 257), (2, 250), (2, 256),
                                     (8, 58), (8, 64)])
def test_worker_moments_each_side_of_the_longest_folded_layer(N, tiles):
    _worker_moments(N, tiles, [tiles * T, 1000, T + 1025, 3, 2049])


def _worker_moments(N, tiles, sizes):
    from oracle import qadam_oracle as oracle
    gcfg, ocfg = configs()
    seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    P, rng = int(seg[-1]), np.random.default_rng(tiles)
    f32 = lambda s: (rng.standard_normal(P) * s).astype(np.float32)  # noqa: E731
    hx, hw = f32(0.02), np.zeros(P, np.float32)
    he, hm, hv = ([np.zeros(P, np.float32) for _ in range(N)] for _ in range(3))
    dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
    x, werr, e, m, v = dev(hx), dev(hw), [dev(a) for a in he], [dev(a) for a in hm], [dev(a) for a in hv]
    q = QAdam(gcfg, seg, N)
    codes = [torch.zeros(q.grad_code_bytes() // 4, dtype=torch.int32, device="cuda") for _ in range(N)]
    scales = [torch.zeros(len(sizes), device="cuda") for _ in range(N)]
    wcodes = torch.zeros(P, dtype=torch.int8, device="cuda")
    for t in (1, 2):
        g = [f32(1e-2) for _ in range(N)]
        q.step_fused_w(t, 1e-3, 0.999, [dev(a) for a in g], m, v, e, codes, scales, x, werr, wcodes)
        torch.cuda.synchronize()
        oracle.step_w(ocfg, seg, t, 1e-3, 0.999, g, he, hm, hv, hx, hw)
    same = lambda d, h: np.array_equal(d.cpu().numpy().view(np.uint32), h.view(np.uint32))  # noqa: E731
    assert same(x, hx) and same(werr, hw)
    for i in range(N):
        assert same(e[i], he[i]) and same(m[i], hm[i]) and same(v[i], hv[i]), i
    q.close()


@pytest.mark.parametrize("k_g", [0, 2, 6])
@pytest.mark.parametrize("n", [1, 33, 255, 257, 4095, 4097, 16383, 16384, 16385, 128 * T + 1, 768 * T, 768 * T + 1, 1024 * T, 1024 * T + 1])
def test_segment_call(n, k_g):
    from oracle import qadam_oracle as oracle
    rng = np.random.default_rng(n)
    g, e = ((rng.standard_normal(n) * s).astype(np.float32) for s in (1e-2, 2e-3))
    g[n // 2] = -0.5                                      # the maximum, away from the ends
    out = oracle.worker_quantize(oracle.OracleConfig(k_g=k_g, k_x=6), [0, n], 0, 1, g, e_want := e.copy())
    words = len(out["words"])
    codes = torch.full((words + 4,), -1, dtype=torch.int32, device="cuda")
    scale, err = torch.full((1,), -1.0, device="cuda"), torch.from_numpy(e).cuda()
    quantize_segment_noalloc(k_g, n, torch.from_numpy(g).cuda(), err, codes, scale)
    assert np.array_equal(codes[:words].cpu().numpy().view(np.uint32), out["words"])
    assert (codes[words:] == -1).all(), "wrote past the segment's code words"
    assert np.array_equal(err.cpu().numpy().view(np.uint32), e_want.view(np.uint32))
    assert np.float32(scale.item()).view(np.uint32) == np.float32(out["scales"][0]).view(np.uint32)


@pytest.mark.parametrize("n", [100, 16384, 16385, 40000])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_segment_call_with_a_non_finite_value(n, bad):
    g = torch.full((n,), 0.25, device="cuda")
    g[n - 1] = float(bad)
    words = (n + 31) // 32 * 3
    codes, scale = torch.full(((words + 3) // 4 * 4,), -1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
    quantize_segment_noalloc(2, n, g, torch.zeros(n, device="cuda"), codes, scale)
    assert not torch.isfinite(scale).item()
    assert (codes == 0).all()
