"""Many-row calibration products and the wide select, at the edges of their
tiles (64 / 128 / 256 output rows, 128 vectors, 32-deep steps) and of the rules
that choose them, against 64-bit products in plain torch."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = 1e-5


def _P():
    import paper_2404_08763_amd as P

    return P


def _layers(d, m, L, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [[(torch.randn((m, d), generator=g, device="cuda") * 0.05).bfloat16() for _ in range(3)] for _ in range(L)]


def _acts64(x, w):
    z = x @ w.double().t()
    return (z / (1 + torch.exp(-z))).abs()


def _rank(n, k):
    return min(max(math.ceil(k * n - 1e-6), 1), n)


# 64-row blocks unless m and N give 80 (128 rows) or 170 (256 rows) blocks of 256
@pytest.mark.parametrize("d,m,N", [
    (8, 7, 1),          # one partial tile of everything
    (40, 300, 129),     # one vector and eight channels past a tile
    (264, 65, 128),     # one neuron past a tile
    (72, 20500, 100),   # 81 blocks: 128 rows
    (64, 11000, 513),   # 215 blocks: 256 rows, one vector past a tile
])
def test_calibrate_threshold_tiles(d, m, N):
    P = _P()
    w = _layers(d, m, 1, 3)[0]
    x = torch.randn((N, d), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda")
    layer = P.Layer(*w)
    ref = _acts64(x.double(), w[0])
    # each product loses 2^-16 of x at most and the sum d roundings; SiLU' is
    # below 1.1; an order statistic moves by no more than its values do
    err = 1.1 * (2.0 ** -16 + d * 2.0 ** -24) * (x.double().abs() @ w[0].double().abs().t()).max().item()
    small = torch.empty(1280 + (N * m * 4 + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    for k in (0.001, 0.5, 0.93, 1.0):
        want = ref.reshape(-1).sort().values[_rank(N * m, k) - 1].item()
        got = P.calibrate_threshold(layer, x, k)
        # a workspace without room for the planes takes the other kernels
        other = P.calibrate_threshold(layer, x, k, ws=small)
        assert abs(got - want) <= err + 4e-6 * want
        assert abs(other - want) <= err + 4e-6 * want


@pytest.mark.parametrize("d,m,N,L", [
    (512, 130, 48, 3),    # two planes
    (512, 65, 33, 2),     # a last group of one row: three planes
    (1032, 693, 35, 3),   # a width without 16-row matrix-core kernels: three planes
    (264, 31, 129, 2),    # fewer neurons than a step is deep
    (2048, 40, 20, 2),    # d > m: the partial sums outgrow the activations
    (256, 5500, 520, 2),  # 256-row blocks, the reduction in parts
])
def test_calibrate_stack_rows(d, m, N, L):
    P = _P()
    ws = _layers(d, m, L, 5)
    stack = P.Stack([P.Layer(*w) for w in ws])
    x0 = torch.randn((N, d), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda")
    got = P.calibrate_stack(stack, x0, 0.5, eps=EPS)
    x = x0.double()
    for l, w in enumerate(ws):
        xn = x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS)
        a = _acts64(xn, w[0])
        want = a.reshape(-1).sort().values[_rank(N * m, 0.5) - 1].item()
        # the bound above, with the stream's own error (the same products, a
        # few 2^-16 of it) on top: twice as much per layer before
        err = (1 + 2 * l) * 1.1 * (2.0 ** -16 + d * 2.0 ** -24) * (xn.abs() @ w[0].double().abs().t()).max().item()
        assert abs(got[l] - want) <= err, (l, got[l], want)
        z = xn @ w[0].double().t()
        x = x + ((z / (1 + torch.exp(-z))) * (xn @ w[1].double().t())) @ w[2].double()
    # the 16-row groups (a workspace of their size) agree within the same error
    groups = max(1280 + (N * m * 4 + 255) // 256 * 256, P.workspace_bytes(d, m, 16)) + 2 * ((N * d * 4 + 255) // 256 * 256)
    other = P.calibrate_stack(stack, x0, 0.5, eps=EPS, ws=torch.empty(groups, dtype=torch.uint8, device="cuda"))
    assert all(abs(a - b) <= 2 * err for a, b in zip(got, other))


def test_calibrate_stack_rows_keeps_inf_and_nan():
    """An infinite channel makes of the vector what it makes of it in fp32: the
    norm in front turns it into NaN."""
    P = _P()
    w = _layers(264, 31, 2, 9)
    x = torch.randn((20, 264), device="cuda")
    x[3, 5] = float("inf")
    t = P.calibrate_stack(P.Stack([P.Layer(*v) for v in w]), x, 1.0, eps=EPS)
    assert all(math.isnan(v) for v in t)  # RMSNorm of an infinity is NaN, the largest bit pattern


@pytest.mark.parametrize("n,shift", [(1, 0), (1, 3), (3, 1), (1023, 2), (16384, 0), (16389, 1), (4200003, 3)])
def test_wide_select_exact(n, shift):
    P = _P()
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(n + 4, generator=g, device="cuda") * torch.exp(3 * torch.randn(n + 4, generator=g, device="cuda"))
    buf[shift + n // 2] = float("inf")
    a = buf[shift:shift + n]  # every alignment of the first value
    s = a.abs().sort().values
    for k in (1e-9, 0.25, 0.5, 0.999, 1.0):
        want = s[_rank(n, k) - 1].item()
        assert P.threshold_from_acts(a, k) == want
        assert P.threshold_from_acts(a, k, ws=torch.empty(1280, dtype=torch.uint8, device="cuda")) == want
    same = torch.full((n,), 0.25, device="cuda")
    assert P.threshold_from_acts(same, 0.5) == 0.25


def test_calibrate_stack_rows_infinite_weight():
    """Three planes: an infinite weight in the second layer leaves the first
    two cutoffs as they are (its neuron's few activations lie above them), and
    everything behind it is NaN, as with the 16-row groups."""
    P = _P()
    d, m, N = 1032, 693, 35
    for which in range(3):
        w = _layers(d, m, 4, 21)
        x = torch.randn((N, d), generator=torch.Generator(device="cuda").manual_seed(22), device="cuda")
        plain = P.calibrate_stack(P.Stack([P.Layer(*v) for v in w]), x, 0.5, eps=EPS)
        w[1][which][5, 7] = math.inf
        stack = P.Stack([P.Layer(*v) for v in w])
        groups = max(1280 + (N * m * 4 + 255) // 256 * 256, P.workspace_bytes(d, m, 16)) + 2 * ((N * d * 4 + 255) // 256 * 256)
        ws = torch.empty(groups, dtype=torch.uint8, device="cuda")
        for t in (P.calibrate_stack(stack, x, 0.5, eps=EPS), P.calibrate_stack(stack, x, 0.5, eps=EPS, ws=ws)):
            assert t[0] == pytest.approx(plain[0], rel=1e-5)
            # (one neuron of 693 moves the middle rank by at most N places)
            assert t[1] == pytest.approx(plain[1], rel=1e-2)
            assert all(math.isnan(v) for v in t[2:])


@pytest.mark.parametrize("d,m,N", [(1032, 31, 2), (512, 31, 3)])
def test_calibrate_stack_rows_three_planes(d, m, N):
    """All 24 bits of x count where three planes are taken (a width or a last
    group of rows that had fp32 products): neighbouring channels of nearly equal
    values meet opposite weights, so an activation is what the low bits differ
    by, 2^-12 of a term.  The norm's and the sums' fp32 roundings are 2^-24 of a
    partial sum of some sqrt(d) = 2^5 terms in 2^5 steps, so about 2^-12 of the
    result and 2^-10 at most; two planes round each x by 2^-19 (root mean
    square), 2^-7 of the result."""
    P = _P()
    g = torch.Generator(device="cuda").manual_seed(d + N)
    r = torch.rand((N, d // 2), generator=g, device="cuda") + 0.5
    x = torch.empty((N, d), device="cuda")
    x[:, 0::2] = r
    x[:, 1::2] = r - r * 2.0 ** -12 * (1 + torch.rand(r.shape, generator=g, device="cuda"))
    half = (torch.randn((m, d // 2), generator=g, device="cuda") * 64).bfloat16()
    wg = torch.empty((m, d), dtype=torch.bfloat16, device="cuda")
    wg[:, 0::2], wg[:, 1::2] = half, -half
    other = (torch.randn((m, d), generator=g, device="cuda") * 0.05).bfloat16()
    stack = P.Stack([P.Layer(wg, other, other)])

    def acts(z):
        return _acts64(z, wg).reshape(-1).sort().values

    xn = x.double() / torch.sqrt((x.double() ** 2).mean(dim=1, keepdim=True) + EPS)
    hi = xn.float().bfloat16().float()
    want, two = acts(xn), acts(hi.double() + (xn.float() - hi).bfloat16().double())
    n = N * m
    got = torch.tensor([P.calibrate_stack(stack, x, (i + 1) / n, eps=EPS)[0] for i in range(n)], dtype=torch.float64,
                       device="cuda")
    err, err2 = ((got - want).norm() / want.norm()).item(), ((two - want).norm() / want.norm()).item()
    print(f"[planes] calibration {d}x{m} N{N}: {err:.2e}, two planes {err2:.2e}")
    assert err <= 2.0 ** -10 and err2 >= 2.0 ** -8
