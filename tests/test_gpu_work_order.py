"""GPU parity at the sizes where the division of the step into work items can go wrong: ends of tiles and of
pieces of tiles, layers of every kind next to each other, and the smallest and largest counts of items."""
import numpy as np
import pytest

from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

# one layer each side of every piece boundary (1024, 2048, 3072, 4096 elements into a tile) behind full tiles
EDGES = [16384 + 4096 * (k % 3) + d for k, d in enumerate([1, 1023, 1024, 1025, 2047, 2048, 2049, 3071, 3073, 4095, 4096])]


@pytest.mark.parametrize("N,rounding,k_g", [(1, 0, 2), (3, 0, 0), (4, 1, 2), (5, 0, 4), (8, 0, 2)])
def test_piece_boundaries(N, rounding, k_g):
    rep, st = _custom(EDGES, N, 3, seed=70 + N, cfgkw=dict(rounding=rounding, k_g=k_g, seed=5), trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


@pytest.mark.parametrize("n", [1, 1023, 1025, 16384, 16385, 4096 * 4095 + 1, 4096 * 4096 + 3])
def test_one_layer_of_each_kind_of_size(n):
    """One-item vectors up to the size from which tiles are cut into fewer pieces."""
    rep, st = _custom([n], 1, 2, seed=90 + n % 97)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()


def test_mixed_layers_off_the_grid():
    sizes = [1001, 70000, 3, 16385, 0, 4096 * 650 + 2, 5, 40001]
    rep, st = _custom(sizes, 2, 3, seed=7, trust=2)
    assert rep.ok() and st == 0 and rep.float_not_bit_exact == 0, rep.line()
