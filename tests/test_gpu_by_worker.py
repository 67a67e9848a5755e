"""GPU parity of the whole-step calls where a large vector makes them one launch per worker and one for the server: on both
sides of the size from which they are, the outputs are those of the separate calls, bit for bit, and on the far side those of
the oracle.  Most of every list is one layer that the chip does not hold, else the step would take a third way (k_parked); the
rules that choose are applied to these lists on the CPU in test_work_split.py."""
import numpy as np
import pytest
import torch

from paper_2004_14180_amd import QAdam
from parity_util import configs
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

N = 4
M = 1 << 20
LAST = {"s": 24 * M, "s off": 48 * M - 1, "w": 32 * M}      # elements up to which the step is one main pass


def sizes_of(kind, more):
    """A long layer and short ones, LAST + more elements; the long one starts on the 16-byte grid or off it."""
    short = [4096 * 700, 1001, 70000, 3, 40001]
    long_one = LAST[kind] + more - sum(short)
    return [short[1], long_one] + short[:1] + short[2:] if kind == "s off" else [long_one] + short


def _bits(t):
    return t.view(torch.int32) if t.dtype == torch.float32 else t


class _State:
    def __init__(self, sizes, w, one_buffer=False, block=0, workers=N, **cfgkw):
        self.cfg, _ = configs(**cfgkw)
        self.workers = N = workers
        seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        P = int(seg[-1])
        gen = torch.Generator(device="cuda")
        gen.manual_seed(P)
        f = lambda s: torch.empty(P, device="cuda").normal_(0.0, s, generator=gen)  # noqa: E731
        self.q = QAdam(self.cfg, seg.tolist(), N)
        self.g, self.e = [f(1e-2) for _ in range(N)], [f(1e-3) for _ in range(N)]
        self.m, self.v = ([f(1e-3) for _ in range(N if w else 1)] for _ in range(2))
        self.v = [t * t for t in self.v]
        self.x, self.werr = f(0.02), f(1e-3)
        self.wcodes = torch.zeros(P, dtype=torch.int8 if self.cfg.k_x <= 6 else torch.int16, device="cuda")
        words = lambda: torch.full((self.q.grad_code_bytes() // 4,), -1, dtype=torch.int32, device="cuda")  # noqa: E731
        self.codes = [words()] * N if one_buffer else [words() for _ in range(N)]
        self.scales = [torch.zeros(len(sizes), device="cuda") for _ in range(N)]
        if block:
            self._move(block, w, P)

    def _move(self, nbytes, w, P):
        """The buffers as qadam_arena_layout deals them to one block."""
        self.block = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        lay = self.q.arena_layout(nbytes, w)
        at = lambda t, o: self.block[o:o + 4 * P].view(torch.float32).copy_(t)  # noqa: E731
        all_at = lambda ts, name: [at(t, o) for t, o in zip(ts, lay[name])]  # noqa: E731
        self.g, self.e = all_at(self.g, "grads"), all_at(self.e, "errs")
        if w:
            self.m, self.v = all_at(self.m, "mw"), all_at(self.v, "vw")
        else:
            self.m, self.v = [at(self.m[0], lay["m"])], [at(self.v[0], lay["v"])]
        self.x, self.werr = at(self.x, lay["x"]), at(self.werr, lay["werr"])

    def step(self, t, w, whole):
        q, N = self.q, self.workers
        if whole and w:
            q.step_fused_w(t, 1e-3, 0.999, self.g, self.m, self.v, self.e, self.codes, self.scales, self.x, self.werr, self.wcodes)
        elif whole:
            q.step_fused(t, 1e-3, 0.999, self.g, self.e, self.codes, self.scales, self.x, self.m[0], self.v[0], self.werr, self.wcodes)
        elif w:
            for i in range(N):
                q.worker_step_w(i, t, 1e-3, 0.999, self.g[i], self.m[i], self.v[i], self.e[i], self.codes[i], self.scales[i])
            q.server_apply_w(t, self.codes, self.scales, self.x)
            q.weight_quantize(t, self.x, self.werr, self.wcodes)
        else:
            for i in range(N):
                q.worker_quantize(i, t, self.g[i], self.e[i], self.codes[i], self.scales[i])
            q.server_step(t, 1e-3, 0.999, self.codes, self.scales, self.x, self.m[0], self.v[0])
            q.weight_quantize(t, self.x, self.werr, self.wcodes)

    def state(self):
        return self.e + self.scales + self.m + self.v + [self.x, self.werr, self.wcodes]


@pytest.mark.parametrize("kind", sorted(LAST))
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("cfgkw", [dict(k_g=2, k_x=6), dict(k_g=0, k_x=14, weight_ef=0), dict(k_g=4, k_x=6, rounding=1, seed=3)])
def test_whole_step_gives_the_bits_of_the_separate_calls(kind, more, cfgkw):
    sizes, w = sizes_of(kind, more), kind == "w"
    a, b = _State(sizes, w, **cfgkw), _State(sizes, w, **cfgkw)
    a.q.profile_enable()
    for t in (1, 2):
        a.step(t, w, True)
        b.step(t, w, False)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
    assert a.q.get_status() == 0
    by_worker = more == 1 and not (w and cfgkw.get("rounding"))
    assert a.q.profile_work() == (sum(sizes), 0, sum(sizes) if by_worker else 0)


def test_a_layer_list_by_worker_against_the_oracle():
    """From the second step on with the filtered scale pass."""
    rep, st = _custom(sizes_of("s", 1), N, 2, seed=41, trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("kind", ["s", "w"])
def test_overlapping_code_buffers_do_not_change_the_step(kind):
    """A caller without use for the codes may pass one buffer for all workers."""
    sizes, w = sizes_of(kind, 1), kind == "w"
    a, b = _State(sizes, w), _State(sizes, w, one_buffer=True)
    a.q.profile_enable(), b.q.profile_enable()
    for t in (1, 2):
        a.step(t, w, True)
        b.step(t, w, True)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state(), b.state())), t
    assert a.q.profile_work()[2] == sum(sizes) and b.q.profile_work()[2] == 0


@pytest.mark.parametrize("kind", ["s", "w"])
def test_buffers_dealt_apart_do_not_change_the_step(kind):
    """One block as qadam_arena_layout deals it, its groups more than 96 GiB apart, where the call is one main pass."""
    torch.cuda.empty_cache()
    nbytes = 200 << 30
    if torch.cuda.mem_get_info()[0] < nbytes + (16 << 30):
        pytest.skip("the device's memory is not free")
    sizes, w = sizes_of(kind, 1), kind == "w"
    a, b = _State(sizes, w), _State(sizes, w, block=nbytes)
    a.q.profile_enable(), b.q.profile_enable()
    for t in (1, 2):
        a.step(t, w, True)
        b.step(t, w, True)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
    assert a.q.profile_work()[2] == sum(sizes) and b.q.profile_work()[2] == 0
    del b                                   # the next tests' handles allocate beside torch
    torch.cuda.empty_cache()
