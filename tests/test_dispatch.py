"""The rules that choose between two kernels for a call, at sizes where both
were timed: the faster one is taken (CPU only; the rules are host functions of
libcats, called by their C++ names)."""
import ctypes

import pytest

import paper_2404_08763_amd as P


def _rule(symbol, *types):
    f = getattr(P.raw(), symbol)
    f.argtypes = list(types)
    f.restype = ctypes.c_bool
    return f


I = ctypes.c_int


# d, partials, rows, us with one column / 16 columns per wave
@pytest.mark.parametrize("d,G,B,one,sixteen", [
    (1032, 64, 1, 6.8, 7.6), (1032, 16, 3, 9.8, 10.4), (512, 64, 3, 8.1, 8.7), (4096, 64, 3, 14.6, 15.3),
    (4096, 8, 1, 7.5, 8.0), (8192, 32, 1, 9.7, 10.4), (3072, 42, 5, 19.9, 20.3),
    (2304, 56, 8, 22.6, 22.0), (4096, 32, 5, 23.1, 22.2), (8192, 16, 8, 39.5, 36.0), (5120, 25, 16, 31.0, 26.8),
    (2048, 64, 16, 21.3, 19.6),
])
def test_sum_of_few_partials(d, G, B, one, sixteen):
    few = _rule("_ZN4cats10reduce_fewEii", I, I)
    assert few(G, B * d) == (sixteen < one)
    assert not few(65, B * d)
