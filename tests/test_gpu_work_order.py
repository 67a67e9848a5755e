"""GPU parity at the sizes where the division of the step into work items can go wrong: ends of tiles and of pieces of
tiles (256 and 512 elements), layers of every size and alignment next to each other, one-item vectors.  The sizes from
which tiles are cut into fewer pieces are test_gpu_many_layers.py's, and test_work_split.py's on the CPU."""
import numpy as np
import pytest

from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

# layers whose last tile ends on, before and behind multiples of 1024, which are boundaries of pieces of either length
EDGES = [16384 + 4096 * (k % 3) + d for k, d in enumerate([1, 1023, 1024, 1025, 2047, 2048, 2049, 3071, 3073, 4095, 4096])]


@pytest.mark.parametrize("N,rounding,k_g", [(1, 0, 2), (3, 0, 0), (4, 1, 2), (5, 0, 4), (8, 0, 2)])
def test_piece_boundaries(N, rounding, k_g):
    rep, st = _custom(EDGES, N, 3, seed=70 + N, cfgkw=dict(rounding=rounding, k_g=k_g, seed=5), trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("N,more", [(3, 400), (5, 220)])
@pytest.mark.parametrize("rounding", [0, 1])
def test_piece_boundaries_with_four_workers_in_flight(N, more, rounding):
    """Behind a layer long enough that the scales come from a launch of their own: the main pass then loads four workers
    at a time, and neither number of workers is a multiple of four."""
    assert (len(EDGES) + more) * N > 1024
    sizes = EDGES[:6] + [255, 257] + EDGES[6:] + [511, 513, 4096 * more]
    rep, st = _custom(sizes, N, 2, seed=60 + N, cfgkw=dict(rounding=rounding, seed=5), trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("n", [1, 1023, 1025, 16384, 16385, 4096 * 4095 + 1, 4096 * 4096 + 3])
def test_one_layer_of_each_kind_of_size(n):
    """From one element to 4097 tiles: both sides of a piece, of the sizes that one workgroup once did, and of 4096 tiles."""
    rep, st = _custom([n], 1, 2, seed=90 + n % 97)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


def test_mixed_layers_off_the_grid():
    sizes = [1001, 70000, 3, 16385, 0, 4096 * 650 + 2, 5, 40001]
    rep, st = _custom(sizes, 2, 3, seed=7, trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()
