"""GPU parity of layers whose scale and quantization are one launch (k_parked): units of every filling, on and off the 16-byte
grid, the longest layer, units that wait for their scale and units put aside, calls on several streams and beside other work,
captured calls, non-finite scales.  The rules that choose are applied to these lists on the CPU in test_work_split.py."""
import time

import numpy as np
import pytest
import torch

from paper_2004_14180_amd import QAdam, QAdamConfig
from test_gpu_by_worker import _State as _AnyState, _bits
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

M, N = 1 << 20, 16
UNIT = 16384
OF_TWO, LONGEST = 256 * UNIT, 1088 * UNIT       # what a launch that holds two units per workgroup serves, what one with three
LEAST = 24 * M // N                     # elements from which the whole step of N workers parks its layers, twice that for stochastic
                                        # rounding; one worker's separate call: 24 M, 64 M


def _State(sizes, w, **kw):
    return _AnyState(sizes, w, workers=N, **kw)


def _sizes(total):
    s = [1, 2047, 2048, 2049, 5, UNIT - 1, UNIT, UNIT + 1, 9 * UNIT - 3, 3, 40 * UNIT + 2050]
    return s + [total - sum(s)]


@pytest.mark.parametrize("polls", [-1, 0])
@pytest.mark.parametrize("less", [0, 1])
@pytest.mark.parametrize("cfgkw", [dict(k_g=2, k_x=6), dict(k_g=0, k_x=14, weight_ef=0), dict(k_g=4, k_x=6, rounding=1, seed=3)])
def test_whole_step_gives_the_bits_of_the_separate_calls(polls, less, cfgkw):
    sizes = _sizes((2 if cfgkw.get("rounding") else 1) * LEAST - less)
    a, b = _State(sizes, False, **cfgkw), _State(sizes, False, **cfgkw)
    a.q.set_scale_polls(polls)
    a.q.profile_enable()
    for t in (1, 2):
        a.step(t, False, True)
        b.step(t, False, False)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
    assert a.q.get_status() == 0
    assert a.q.profile_work()[0] == (sum(sizes) if less else 0)


@pytest.mark.parametrize("polls", [1, 2, 4])
def test_some_units_of_a_layer_are_put_aside(polls):
    """Few polls: some workgroups of a layer quantize the units they hold while others put theirs aside and load them again.  The
    layers have more than eight units, whose workgroups poll several copies of the scale."""
    sizes = [LEAST // 8, 40 * UNIT + 77, 20 * UNIT + 1, 9 * UNIT]
    sizes.append(LEAST - sum(sizes))
    a, b = _State(sizes, False), _State(sizes, False)
    a.q.set_scale_polls(polls)
    for t in (1, 2, 3):
        a.step(t, False, True)
        b.step(t, False, False)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t


# sizes, workers, trust, elements whose scales have a pass of their own
ORACLE = [([OF_TWO, 2 * M, 1001, 0, 70001, 2 * M], 1, 0, 0),                    # two units, all parked, an empty layer
          ([OF_TWO, 2 * M, 1001, 0, 2 * M - 1002], 1, 0, 8 * M - 1),            # not enough of them
          ([700 * UNIT, 0, OF_TWO + 3, 77], 1, 0, 0),                           # three units, all parked
          ([OF_TWO + 1, 8 * M - 9, 7], 1, 0, 12 * M - 1),                       # not enough of them
          ([LONGEST + 1, 3, OF_TWO, OF_TWO, OF_TWO - 5, 77], 4, 2, LONGEST + 1),        # two units, beside a longer layer, filtered
          ([LONGEST + 1, 3, LONGEST - 1, 2 * M], 3, 2, LONGEST + 1)]                    # three


@pytest.mark.parametrize("sizes,workers,trust,scanned", ORACLE)
def test_against_the_oracle(sizes, workers, trust, scanned):
    work = []
    rep, st = _custom(sizes, workers, 2, seed=43, trust=trust, work=work)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()
    assert [w[:2] for w in work] == [(scanned, 0), (scanned, scanned if trust else 0)]


class _Calls:
    """worker_quantize for every worker, whose layers one worker's call parks."""

    def __init__(self, sizes, workers=2):
        seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        self.workers, self.q = workers, QAdam(QAdamConfig(), seg, workers)
        q = self.q
        gen = torch.Generator(device="cuda")
        gen.manual_seed(5)
        P = int(seg[-1])
        f = lambda s: torch.empty(P, device="cuda").normal_(0.0, s, generator=gen)  # noqa: E731
        self.g, self.e = [f(1e-2) for _ in range(workers)], [f(1e-3) for _ in range(workers)]
        self.codes = [torch.full((q.grad_code_bytes() // 4,), -1, dtype=torch.int32, device="cuda") for _ in range(workers)]
        self.scales = [torch.zeros(len(sizes), device="cuda") for _ in range(workers)]
        torch.cuda.synchronize()

    def run(self, streams, steps=3, beside=None):
        """Seconds; beside: enqueues work on another stream before every step."""
        t0 = time.perf_counter()
        for t in range(1, steps + 1):
            if beside:
                beside()
            for i in range(self.workers):
                self.q.worker_quantize(i, t, self.g[i], self.e[i], self.codes[i], self.scales[i], stream=streams[i])
        torch.cuda.synchronize()
        assert self.q.get_status() == 0
        return time.perf_counter() - t0

    def state(self):
        return self.e + self.codes + self.scales


SIZES = [2 * M] * 11 + [1003, 2 * M]     # a separate call parks from 24 M on


def _matmuls():
    a, stream = torch.randn(4096, 4096, device="cuda", dtype=torch.bfloat16), torch.cuda.Stream()

    def run():
        with torch.cuda.stream(stream):
            for _ in range(8):
                torch.matmul(a, a)
    torch.cuda.synchronize()
    return run


def test_workers_on_two_streams():
    one, two, beside = _Calls(SIZES), _Calls(SIZES), _Calls(SIZES)
    one.run([torch.cuda.current_stream()] * 2)
    two.run([torch.cuda.Stream() for _ in range(2)])
    beside.run([torch.cuda.Stream() for _ in range(2)], beside=_matmuls())
    assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(one.state(), two.state()))
    assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(one.state(), beside.state()))


def test_calls_on_two_streams_do_not_wait_for_workgroups_without_a_place():
    """The workgroups of two calls share the chip, so that half of each call's have no place yet.  Where the others waited for
    them, and then read whole layers to find the scale, a call took twelve times as long as alone; it takes about as long, and
    twice as long is more than any run of one side differs."""
    c = _Calls([768 * 768, 3 * 768 * 768, 768, 4 * 768 * 768, 4 * 768 * 768, 768] * 12)
    one, two = [torch.cuda.current_stream()] * 2, [torch.cuda.Stream() for _ in range(2)]
    c.run(one), c.run(two)
    alone, beside = (min(c.run(streams, 10) for _ in range(3)) for streams in (one, two))
    assert beside < 2.0 * alone, (alone, beside)


ON_FOUR_STREAMS = [[768 * UNIT, 768 * UNIT + 5], [1003, 1024 * UNIT, 1024 * UNIT, 300 * UNIT]]


@pytest.mark.parametrize("sizes", ON_FOUR_STREAMS)
def test_long_layers_on_four_streams_find_the_units_without_a_workgroup(sizes):
    """Three of four launches have a part of their workgroups on the chip, and a layer needs units that no workgroup has begun with.
    Where every workgroup looked for the first of them, a call took 1.5 to 1.6 times as long as alone; it takes up to 1.25
    times as long.  The bits are those of calls one after the other."""
    one, many = _Calls(sizes, 4), _Calls(sizes, 4)
    alone, beside = [torch.cuda.current_stream()] * 4, [torch.cuda.Stream() for _ in range(4)]
    one.run(alone), many.run(beside)
    assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(one.state(), many.state()))
    a, b = (min(one.run(streams, 10) for _ in range(4)) for streams in (alone, beside))
    assert b < 1.42 * a, (a, b)


def test_overlapping_code_buffers_do_not_change_the_step():
    """A caller without use for the codes may pass one buffer for all workers, whose layers are then not parked."""
    sizes = _sizes(LEAST)
    a, b = _State(sizes, False), _State(sizes, False, one_buffer=True)
    for t in (1, 2):
        a.step(t, False, True)
        b.step(t, False, True)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state(), b.state())), t


def test_captured_step_is_the_eager_one():
    sizes = _sizes(LEAST)
    a, b = _State(sizes, False), _State(sizes, False)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        a.step(1, False, True)
    for t in (1, 2, 3):
        graph.replay()
        b.step(1, False, True)
        torch.cuda.synchronize()
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t


@pytest.mark.parametrize("polls", [-1, 0])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_scale_that_is_not_finite_stays_in_its_layer(polls, bad):
    sizes = _sizes(LEAST)
    a, b = _State(sizes, False), _State(sizes, False)
    a.q.set_scale_polls(polls)
    at = sum(sizes[:8]) + 5 * UNIT                       # in the layer of nine units
    for s in (a, b):
        s.g[3][at] = bad
    a.step(1, False, True)
    b.step(1, False, False)
    assert a.q.get_status() == b.q.get_status() == 1
    for p, r in zip(a.codes + a.scales, b.codes + b.scales):
        assert torch.equal(_bits(p), _bits(r))
    lo, hi = sum(sizes[:8]), sum(sizes[:9])
    for p, r in zip(a.e, b.e):
        assert torch.equal(_bits(p[:lo]), _bits(r[:lo])) and torch.equal(_bits(p[hi:]), _bits(r[hi:]))


def test_polls_are_checked():
    q = QAdam(QAdamConfig(), [0, 10], 1)
    with pytest.raises(Exception):
        q.set_scale_polls(-2)
    q.set_scale_polls(2**31 - 1)            # accepted, as many as end in a bounded time are used


@pytest.mark.parametrize("polls", [-1, 0, 3])
@pytest.mark.parametrize("sizes", [[256 * UNIT + 1, 1001, 130 * UNIT - 5, 2047, 300 * UNIT],    # just beyond what two units serve
                                   [1001, 1088 * UNIT]])                                        # the longest, off the grid
@pytest.mark.parametrize("cfgkw", [dict(k_g=2, k_x=6), dict(k_g=4, k_x=6, rounding=1, seed=3)])
def test_lists_whose_workgroups_hold_three_units(polls, sizes, cfgkw):
    a, b = (_AnyState(sizes, False, workers=5, **cfgkw) for _ in range(2))
    a.q.set_scale_polls(polls)
    a.q.profile_enable()
    for t in (1, 2):
        a.step(t, False, True)
        b.step(t, False, False)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
    assert a.q.get_status() == 0
    assert a.q.profile_work()[0] == 0       # every layer was parked


@pytest.mark.parametrize("polls", [-1, 0, 3])
@pytest.mark.parametrize("sizes,workers", [(_sizes(9 * M // 2), N),                             # 72 M, units of every filling
                                           ([256 * UNIT + 1, 1001, 130 * UNIT - 5, 2047, 300 * UNIT], 8),   # three units
                                           ([1001, 1088 * UNIT], 8)])                           # the longest, off the grid
@pytest.mark.parametrize("cfgkw", [dict(k_g=2, k_x=6), dict(k_g=0, k_x=14, weight_ef=0, adam_flavor=1),
                                   dict(k_g=4, k_x=6, rounding=1, seed=3)])
def test_variant_w_gives_the_bits_of_the_separate_calls(polls, sizes, workers, cfgkw):
    """Units put aside find their local moments advanced when they are loaded again."""
    a, b = (_AnyState(sizes, True, workers=workers, **cfgkw) for _ in range(2))
    a.q.set_scale_polls(polls)
    a.q.profile_enable()
    for t in (1, 2):
        a.step(t, True, True)
        b.step(t, True, False)
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
    assert a.q.get_status() == 0
    assert a.q.profile_work()[0] == 0


W_CALL = [36 * UNIT - 7] * 86 + [0, 3]
W_CALL_OF_THREE = [2000 * UNIT, 1088 * UNIT] + [1024 * UNIT] * 4 + [5]         # beside a longer layer


@pytest.mark.parametrize("sizes", [W_CALL, W_CALL_OF_THREE])
def test_variant_w_one_workers_call(sizes):
    """One worker's call that parks its layers, against plain tensor operations: moments and scales bit for bit, residuals within
    half the widest gap of the grid."""
    a, b = _AnyState(sizes, True, workers=1), _AnyState(sizes, True, workers=1)
    for t in (1, 2):
        a.step(t, True, False)
        g, m, v = b.g[0], b.m[0], b.v[0]
        f = lambda c: torch.tensor(c, dtype=torch.float32, device="cuda")  # noqa: E731
        b1, b2, one = f(0.9), f(0.999), f(1.0)
        v.copy_((b2 * v) + ((one - b2) * (g * g)))
        m.copy_((b1 * m) + ((one - b1) * g))
        assert torch.equal(_bits(a.v[0]), _bits(v)) and torch.equal(_bits(a.m[0]), _bits(m)), t
        p = (f(1e-3) * m) / torch.sqrt(v + f(b.cfg.eps)) + b.e[0]
        at = 0
        for l, n in enumerate(sizes):
            assert a.scales[0][l] == (p[at:at + n].abs().max() if n else 0.0), (t, l)
            at += n
        b.e[0].copy_(a.e[0])        # every next step begins from the same state
        assert (a.e[0].abs() <= 0.2501 * a.scales[0].repeat_interleave(torch.tensor(sizes, device="cuda"))).all()


def beside_longer(sizes):
    """The list with a layer behind it that keeps variant W from parking any of them."""
    return sizes + [2 * sum(sizes) + 1]


W_CALLS = [(W_CALL, 0), (W_CALL_OF_THREE, 0), ([36 * UNIT - 7] * 130 + [1, 2050], 1), ([1001] + [1024 * UNIT] * 5, 1)]


@pytest.mark.parametrize("streams", [1, 2])
@pytest.mark.parametrize("polls", [-1, 3])
@pytest.mark.parametrize("sizes,rounding", W_CALLS)
def test_variant_w_calls_give_the_bits_of_two_passes(sizes, rounding, polls, streams):
    """Two workers' calls, one after the other and on streams of their own, against those of a list whose first layers are the same and
    are not parked."""
    a, b = (_AnyState(s, True, workers=2, rounding=rounding, seed=3) for s in (sizes, beside_longer(sizes)))
    P, L = sum(sizes), len(sizes)
    a.q.set_scale_polls(polls)
    for i in range(2):
        for p, r in ((a.g, b.g), (a.e, b.e), (a.m, b.m), (a.v, b.v)):
            r[i][:P].copy_(p[i])
    on = [torch.cuda.Stream() for _ in range(2)] if streams == 2 else [torch.cuda.current_stream()] * 2
    torch.cuda.synchronize()
    for t in (1, 2):
        for s, where in ((a, on), (b, [None, None])):
            for i in (1, 0):
                s.q.worker_step_w(i, t, 1e-3, 0.999, s.g[i], s.m[i], s.v[i], s.e[i], s.codes[i], s.scales[i], stream=where[i])
        torch.cuda.synchronize()
        for i in range(2):
            for name, p, r in (("e", a.e, b.e), ("m", a.m, b.m), ("v", a.v, b.v)):
                assert torch.equal(_bits(p[i]), _bits(r[i][:P])), (t, name, i)
            assert torch.equal(_bits(a.scales[i]), _bits(b.scales[i][:L])), (t, i)
            assert torch.equal(a.codes[i], b.codes[i][:a.codes[i].numel()]), (t, i)
    assert a.q.get_status() == b.q.get_status() == 0


@pytest.mark.parametrize("sizes", [_sizes(40 * M // N), [1001, 300 * UNIT, 20 * UNIT]])    # two units, three
def test_captured_step_of_variant_w_is_the_eager_one(sizes):
    w = N if sizes[0] == 1 else 2 * N
    a, b = (_AnyState(sizes, True, workers=w) for _ in range(2))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        a.step(1, True, True)
    for t in (1, 2, 3):
        graph.replay()
        b.step(1, True, True)
        torch.cuda.synchronize()
        assert all(torch.equal(_bits(p), _bits(r)) for p, r in zip(a.state() + a.codes, b.state() + b.codes)), t
