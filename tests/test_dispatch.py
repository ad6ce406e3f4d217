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


# d, partials, blocks that listed the neurons, rows, us with one column / 16 columns per wave
@pytest.mark.parametrize("d,G,Gseg,B,one,sixteen", [
    (1032, 64, 64, 1, 6.8, 7.6), (1032, 16, 16, 3, 9.8, 10.4), (512, 64, 64, 3, 8.1, 8.7), (4096, 64, 64, 3, 14.6, 15.3),
    (4096, 8, 8, 1, 7.5, 8.0), (8192, 32, 32, 1, 9.7, 10.4), (3072, 42, 256, 5, 19.9, 20.3),
    (2560, 47, 256, 6, 22.2, 22.8), (8192, 20, 20, 2, 14.7, 15.0), (4096, 32, 256, 4, 50.9, 50.4),
    (4104, 20, 20, 4, 17.2, 16.8), (2048, 47, 256, 9, 20.8, 19.6), (2304, 56, 256, 8, 22.6, 22.0),
    (4096, 32, 256, 5, 23.1, 22.2), (8192, 16, 256, 8, 39.5, 36.0), (5120, 25, 256, 16, 31.0, 26.8),
    (2048, 64, 256, 16, 21.3, 19.6),
])
def test_sum_of_few_partials(d, G, Gseg, B, one, sixteen):
    few = _rule("_ZN4cats10reduce_fewEiii", I, I, I)
    assert few(G, Gseg, B * d) == (sixteen < one)
    assert not few(65, 256, B * d)


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("B", [3, 8, 9, 16])
def test_gateup_tiles(B, dense):
    """The tiles of a gate/up step: instantiated, no more rounds than the
    largest step needs, and within the neurons a block's LDS arrays hold."""
    f = P.raw()._ZN4cats12gateup_tilesEiib
    f.argtypes = [I, I, ctypes.c_bool]
    for m in (1, 255, 256, *range(257, 65537, 37), 65536):
        nb = -(-m // min(m, 256))
        T = f(m, B, dense)
        most = 6 if B > 8 else 8
        assert T in ((2, 4, 6, 8) if dense else (1, 2, 3, 4, 6, 8)) and T <= most
        cols = 16 * T // (2 if dense else 1)
        rounds = -(-nb // cols)
        assert rounds == -(-nb // (16 * most // (2 if dense else 1)))
        if not dense and T <= 4:
            assert rounds == 1 or (T == 4 and nb <= 128)
    # rows of x, neurons, tiles a step where both were timed
    for rows, m, d_, T in ((9, 28672, False, 4), (16, 28672, False, 4), (8, 28672, False, 8), (9, 14336, True, 4),
                           (4, 20000, True, 6), (8, 34000, False, 6)):
        assert f(m, rows, d_) == T


# d, m, dense, us with k_mlp_gateup / with x in registers
@pytest.mark.parametrize("d,m,dense,stream,narrow", [
    (512, 3000, False, 15.4, 15.7), (512, 5632, False, 18.4, 17.6), (512, 28672, False, 34.6, 29.2),
    (512, 60000, False, 59.0, 46.4), (1024, 5632, False, 19.3, 19.9), (1024, 8000, False, 23.6, 22.5),
    (1024, 11008, False, 26.8, 23.7), (1024, 28672, False, 49.8, 43.0), (2048, 28672, False, 67.7, 70.0),
    (2048, 34000, False, 86.2, 80.7),
    (512, 11008, True, 19.3, 19.5), (512, 28672, True, 35.4, 30.6), (1024, 8000, True, 20.1, 21.2),
    (1024, 18000, True, 33.0, 31.0), (2048, 28672, True, 66.6, 70.9),
])
def test_gateup_of_narrow_blocks(d, m, dense, stream, narrow):
    f = _rule("_ZN4cats13gateup_narrowEiib", I, I, ctypes.c_bool)
    assert f(d, m, dense) == (narrow < stream)
    # x in registers pipelines from one of a block's tiles to the next
    assert not narrow < stream or m // 256 > 16
    for other in (d + 8, d - 8, 3072, 5120):  # widths that it has no instance for
        assert not f(other, m, dense)


# d, m, rows, dense, us with the fused kernel / on the matrix cores
@pytest.mark.parametrize("d,m,B,dense,fused,mfma", [
    (4096, 11008, 2, False, 40, 45), (4096, 11008, 3, False, 49.0, 50.3), (8192, 28672, 3, False, 251, 208),
    (6144, 2000, 3, False, 44.1, 33.8), (8192, 512, 3, False, 36.2, 34.7), (5640, 128, 3, False, 26.9, 29.3),
    (8192, 512, 4, True, 41.9, 25.3), (4096, 11008, 4, False, 54.0, 52.1), (1024, 28000, 4, False, 58, 45),
    (2856, 20000, 4, False, 78, 86), (4096, 34000, 4, False, 135, 146), (4096, 34000, 4, True, 140, 139),
    (2048, 34000, 4, False, 84, 87), (1024, 34000, 4, False, 67, 56),
    (256, 2000, 8, True, 14.2, 13.9), (256, 2000, 5, True, 12.6, 13.8), (520, 4000, 5, True, 18.6, 16.0),
    (256, 2000, 8, False, 13.7, 15.6), (64, 3000, 6, False, 13.3, 14.4), (256, 3000, 6, False, 14.0, 15.5),
    (512, 2000, 8, False, 14.8, 16.7), (136, 4000, 8, False, 17.4, 15.5), (1000, 2000, 5, False, 16.3, 18.4),
    (1024, 2000, 5, False, 15.5, 16.8), (1000, 4000, 5, False, 19.3, 19.2), (776, 2000, 6, False, 16.4, 18.1),
    (776, 2500, 6, False, 18.4, 17.8), (1032, 2000, 6, False, 20.2, 19.3), (776, 3000, 5, False, 17.1, 17.9),
    (1032, 1000, 8, False, 23.3, 18.6), (776, 2000, 8, False, 19.4, 18.3), (2056, 1000, 5, False, 27.7, 21.6),
    (256, 3000, 9, False, 23.8, 15.6), (8192, 28672, 8, True, 587, 224),
])
def test_batched_rows(d, m, B, dense, fused, mfma):
    f = _rule("_ZN4cats12batched_rowsEiiib", I, I, I, ctypes.c_bool)
    assert f(d, m, B, dense) == (mfma < fused)


@pytest.mark.parametrize("B", [5, 8, 9, 16])
@pytest.mark.parametrize("d,m", [(1032, 693), (264, 1000), (8, 65536), (4104, 100)])
def test_small_three_plane_blocks_stay_fused(d, m, B):
    """Where the forward is bit for bit the separate kernels' result."""
    f = _rule("_ZN4cats12batched_rowsEiiib", I, I, I, ctypes.c_bool)
    if B * m * max(d, 512) <= 8_000_000:
        assert not f(d, m, B, False) and not f(d, m, B, True)
