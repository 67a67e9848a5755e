"""The binding's buffer checks: every buffer of a call is refused or taken on its own, whatever its place in the list."""
import numpy as np
import pytest
import torch

from paper_2004_14180_amd import QAdam, binding
from paper_2004_14180_amd.binding import _stream
from parity_util import configs

pytestmark = pytest.mark.gpu

P, N = 4100, 3


def _call(q, codes_dtype=torch.int32, **put):
    """One fused step on fresh buffers; put = {name: tensor in the place of the last buffer of that name}."""
    torch.manual_seed(0)
    f = lambda n: torch.randn(n, device="cuda")  # noqa: E731
    b = dict(grads=[f(P) for _ in range(N)], errs=[torch.zeros(P, device="cuda") for _ in range(N)],
             codes=[torch.zeros(q.grad_code_bytes(), dtype=torch.int8, device="cuda").view(codes_dtype) for _ in range(N)],
             scales=[torch.zeros(2, device="cuda") for _ in range(N)])
    s = dict(x=f(P), m=torch.zeros(P, device="cuda"), v=torch.zeros(P, device="cuda"),
             werr=torch.zeros(P, device="cuda"), wcodes=torch.zeros(P, dtype=torch.int8, device="cuda"))
    for name, t in put.items():
        if name in b:
            b[name][-1] = t
        else:
            s[name] = t
    q.step_fused(1, 1e-3, 0.999, **b, **s)
    return b, s


@pytest.mark.parametrize("name", ["grads", "errs", "scales", "x", "werr"])
@pytest.mark.parametrize("bad", ["none", "host", "double", "short", "strided", "integer"])
def test_refused(name, bad):
    q = QAdam(configs()[0], np.array([0, 1000, P]), N)
    n = 2 if name == "scales" else P
    t = {"none": None, "host": torch.zeros(n), "double": torch.zeros(n, dtype=torch.float64, device="cuda"),
         "short": torch.zeros(n - 1, device="cuda"), "strided": torch.zeros(2 * n, device="cuda")[::2],
         "integer": torch.zeros(n, dtype=torch.int32, device="cuda")}[bad]
    with pytest.raises(ValueError, match=name):
        _call(q, **{name: t})
    q.close()


@pytest.mark.parametrize("dtype", [torch.int8, torch.uint8, torch.int16, torch.int64])
def test_codes_of_any_integer_type(dtype):
    q = QAdam(configs()[0], np.array([0, 1000, P]), N)
    (a, sa), (b, sb) = _call(q), _call(q, codes_dtype=dtype)
    for i in range(N):
        assert torch.equal(a["codes"][i], b["codes"][i].view(torch.int32))
    assert torch.equal(sa["x"], sb["x"])
    with pytest.raises(ValueError, match="codes"):
        _call(q, codes=torch.zeros(q.grad_code_bytes() // 4 - 1, dtype=torch.int32, device="cuda"))
    with pytest.raises(ValueError, match="codes"):
        _call(q, codes=torch.zeros(q.grad_code_bytes(), device="cuda"))
    q.close()


def test_the_current_stream_is_used():
    s = torch.cuda.Stream()
    assert _stream(None) == (torch.cuda.current_stream().cuda_stream or None)
    with torch.cuda.stream(s):
        assert _stream(None) == s.cuda_stream
    assert _stream(s) == s.cuda_stream


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("form", ["parameter", "subclass", "tuple", "generator-made list", "longer", "numpy numbers", "a stream", "no native part"])
def test_other_forms_give_the_common_forms_result(form, monkeypatch):
    """What the native calls do not take goes through the checks in Python, with the same outcome."""
    q = QAdam(configs()[0], np.array([0, 1000, P]), N)

    def step(put):
        torch.manual_seed(0)
        f = lambda n: torch.randn(n, device="cuda")  # noqa: E731
        g, e = [f(P) for _ in range(N)], [torch.zeros(P, device="cuda") for _ in range(N)]
        c = [torch.zeros(q.grad_code_bytes() // 4, dtype=torch.int32, device="cuda") for _ in range(N)]
        s = [torch.zeros(2, device="cuda") for _ in range(N)]
        x, m, v, w = f(P), torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda"), torch.zeros(P, device="cuda")
        wc, lr, stream = torch.zeros(P, dtype=torch.int8, device="cuda"), 1e-3, None
        if put == "parameter":
            g = [torch.nn.Parameter(t) for t in g]
        elif put == "subclass":
            g[1] = g[1].as_subclass(_Sub)
        elif put == "tuple":
            g, s = tuple(g), tuple(s)
        elif put == "generator-made list":
            g = list(t for t in g)
        elif put == "longer":
            g[0] = torch.cat([g[0], f(5)])
        elif put == "numpy numbers":
            lr = np.float64(lr)
        elif put == "a stream":
            torch.cuda.synchronize()
            stream = torch.cuda.Stream()
        elif put == "no native part":
            monkeypatch.setattr(binding, "_native", binding._Unavailable())
        q.step_fused(1, lr, 0.999, g, e, c, s, x, m, v, w, wc, stream=stream)
        torch.cuda.synchronize()
        monkeypatch.undo()
        assert not isinstance(binding._native, binding._Unavailable)
        return e + c + list(s) + [x, m, v, w, wc]

    assert all(torch.equal(a, b) for a, b in zip(step(form), step(None)))
    q.close()
    with pytest.raises(Exception):
        step(None)                      # a closed handle stays refused
