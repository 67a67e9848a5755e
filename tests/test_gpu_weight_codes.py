"""Weight quantizer and decoder at the lengths where a wavefront's share of the vector ends."""
import numpy as np
import pytest
import torch

from oracle import qadam_oracle as oracle
from paper_2004_14180_amd import QAdam
from parity_util import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_x,weight_ef,rounding", [(6, 1, 0), (14, 0, 0), (14, 1, 1)])
@pytest.mark.parametrize("n", [1, 3, 7, 9, 255, 256, 257, 511, 513, 2051, 70001])
def test_lengths(n, k_x, weight_ef, rounding):
    gcfg, ocfg = configs(k_x=k_x, weight_ef=weight_ef, rounding=rounding)
    rng = np.random.default_rng(n)
    x = rng.uniform(-0.55, 0.55, n).astype(np.float32)
    werr = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    want_err = werr.copy()
    want = oracle.weight_quantize(ocfg, 3, x, want_err)
    q = QAdam(gcfg, [0, n], 1)
    guard = 16                                            # elements behind the end that must stay as they are
    wt = torch.int8 if k_x <= 6 else torch.int16
    err = torch.from_numpy(np.concatenate([werr, np.full(guard, 7, np.float32)])).cuda()
    wc = torch.full((n + guard,), 77, dtype=wt, device="cuda")
    full = torch.full((n + guard,), 7.0, device="cuda")
    half = torch.full((n + guard,), 7.0, dtype=torch.float16, device="cuda")
    q.weight_quantize(3, torch.from_numpy(x).cuda(), err[:n], wc[:n])
    q.weight_dequantize(wc[:n], full[:n])
    q.weight_dequantize_f16(wc[:n], half[:n])
    assert np.array_equal(wc[:n].cpu().numpy(), want["wcodes"])
    assert np.array_equal(err[:n].cpu().numpy(), want_err)
    assert np.array_equal(full[:n].cpu().numpy(), want["xhat"])
    assert np.array_equal(half[:n].cpu().numpy(), want["xhat"].astype(np.float16))
    assert (wc[n:] == 77).all() and (err[n:] == 7).all() and (full[n:] == 7).all() and (half[n:] == 7).all()
    q.close()


@pytest.mark.parametrize("k_x,half", [(6, False), (6, True), (14, False), (14, True)])
def test_decoder_each_side_of_its_rule(k_x, half):
    """The vector lengths on both sides of the two lines between the decoder's launch shapes (6 MiB, and 160 or 40 MiB of
    codes and output), each with a ragged end."""
    size = (1 if k_x <= 6 else 2) + (2 if half else 4)
    for line in (6 << 20, (40 if half and k_x > 6 else 160) << 20):
        for n in (line // size, line // size + 1, line // size + 4099):
            q = QAdam(configs(k_x=k_x)[0], [0, n], 1)
            wt, top = (torch.int8, 64) if k_x <= 6 else (torch.int16, 1 << 14)
            wc = torch.randint(-top, top + 1, (n,), dtype=wt, device="cuda")
            out = torch.full((n + 16,), 7.0, dtype=torch.float16 if half else torch.float32, device="cuda")
            (q.weight_dequantize_f16 if half else q.weight_dequantize)(wc, out[:n])
            want = (wc.to(torch.float32) * 2.0 ** -(k_x + 1)).to(out.dtype)      # exact, then one rounding
            assert torch.equal(out[:n], want) and (out[n:] == 7).all(), n
            q.close()


@pytest.mark.parametrize("k_x,weight_ef,rounding", [(6, 1, 0), (14, 1, 1), (14, 0, 0)])
def test_quantizer_each_side_of_its_rule(k_x, weight_ef, rounding):
    """The vector lengths on both sides of the two lines between the weight quantizer's launch shapes (16 and 96 MiB of
    weights, residual and codes), each with a ragged end."""
    size = 8 + (1 if k_x <= 6 else 2)
    gcfg, ocfg = configs(k_x=k_x, weight_ef=weight_ef, rounding=rounding)
    for line in (16 << 20, 96 << 20):
        for n in (line // size - 1, line // size + 1, line // size + 4099):
            rng = np.random.default_rng(n)
            x = rng.uniform(-0.55, 0.55, n).astype(np.float32)
            werr = (rng.standard_normal(n, dtype=np.float32) * np.float32(1e-3))
            q = QAdam(gcfg, [0, n], 1)
            err = torch.from_numpy(np.concatenate([werr, np.full(16, 7, np.float32)])).cuda()
            wc = torch.full((n + 16,), 77, dtype=torch.int8 if k_x <= 6 else torch.int16, device="cuda")
            q.weight_quantize(3, torch.from_numpy(x).cuda(), err[:n], wc[:n])
            want = oracle.weight_quantize(ocfg, 3, x, werr)
            assert np.array_equal(wc[:n].cpu().numpy(), want["wcodes"]) and np.array_equal(err[:n].cpu().numpy(), werr), n
            assert (wc[n:] == 77).all() and (err[n:] == 7).all(), n
            q.close()
