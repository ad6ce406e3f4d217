"""The matrix-core path for 3..16 rows at the edges of its tiles and splits,
against 64-bit products in plain torch: neuron tiles of 1..8 per block and more
than one round of them, 8- and 16-row operands, two and three planes of x,
widths that end inside a 64-column step, lists, and RMSNorm in front."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = 1e-5
TWO_PLANES = (512, 1024, 2048, 3072, 4096, 5120)
SHAPES = [
    (512, 7, 16),        # one-neuron blocks, two planes
    (512, 5000, 8),      # two tiles
    (1024, 700, 9),
    (8192, 600, 8),      # one tile, the widest rows
    (1032, 3000, 5),     # a width that ends inside a step
    (2856, 7001, 11),
    (136, 12000, 8),     # three tiles, fewer steps than waves
    (136, 16000, 16),    # four tiles, 16-row operands
    (200, 23000, 13),    # six tiles
    (72, 33000, 6),      # more than eight tiles: a second round
    (8192, 600, 3),      # the fewest rows, wide
    (5128, 700, 4),
    (2048, 14000, 4),    # three planes at a width that has two from 5 rows
    (5128, 7000, 4),     # up to four rows: two tiles, then three, six and eight
    (6152, 11500, 3),
    (1088, 23100, 4),
    (1024, 28000, 4),
    (8, 65536, 5),       # the most neurons, the narrowest rows
    (264, 28672, 16),    # seven tiles: two rounds of four (dense: three of three)
    (1088, 28700, 9),    # eight tiles less fifteen neurons
    (136, 17000, 8),     # five tiles (dense: two rounds of three)
    (136, 34000, 12),    # nine tiles: two rounds of six
    (512, 9001, 6),      # x in registers: three tiles, a ragged last one
    (1024, 8000, 16),    # its fewest neurons at 1024 columns
    (512, 12300, 9),     # its fewest dense ones
    (1024, 28672, 5),
    (2048, 32800, 7),    # its widest, CATS only, more than eight tiles
    (512, 65536, 16),    # the most neurons
    (2048, 1000, 8),     # the sum of few partials by 16 columns per wave, at its fewest outputs
    (2040, 1000, 8),     # and by one column, at nearly its most
]


def _P():
    import paper_2404_08763_amd as P

    return P


def _silu(z):
    return z / (1 + torch.exp(-z))


def _inputs(d, m, B, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = [(torch.randn((m, d), generator=g, device="cuda") * 0.05).bfloat16() for _ in range(3)]
    return w, torch.randn((B, d), generator=g, device="cuda"), torch.randn((B, d), generator=g, device="cuda")


def _gap(mag, k):
    """A cutoff in the widest gap near the k-quantile: rounding decides no mask."""
    s = mag.reshape(-1).sort().values
    n = s.numel()
    lo, hi = int(n * max(k - 0.02, 0)), min(int(n * (k + 0.02)) + 2, n - 1)
    i = int(torch.argmax((s[lo + 1:hi + 1] - s[lo:hi]) / s[lo + 1:hi + 1])) + lo
    return float(((s[i] + s[i + 1]) / 2).float())


def _bound(d, B):
    # two planes lose 2^-17 of each x and h (relative, random in sign); three
    # lose nothing and the fp32 sums a few 2^-24 of the result
    return 2.0 ** -15 if d in TWO_PLANES and B >= 5 else 2.0 ** -18


@pytest.mark.parametrize("d,m,B", SHAPES)
def test_batched_shapes(d, m, B):
    P = _P()
    w, x, res = _inputs(d, m, B, d + m + B)
    layer = P.Layer(*w)
    ws = P.workspace(d, m, B)
    g, u = (x.double() @ w[i].double().t() for i in range(2))
    v = _silu(g)
    for k in (0.5, 0.9):
        t = _gap(v.abs(), k)
        keep = v.abs() >= t
        want = res.double() + torch.where(keep, v * u, torch.zeros_like(v)) @ w[2].double()
        ws.random_(0, 256)  # the workspace may hold anything
        y, aux = P.mlp_forward(layer, x, t, residual=res, ws=ws, aux=True)
        assert torch.equal(y, P.mlp_forward(layer, x, t, residual=res, ws=ws))
        assert ((y.double() - want).norm() / want.norm()).item() <= _bound(d, B)
        for b in range(B):
            idx = keep[b].nonzero()[:, 0]
            n = int(aux["cnt"][b])
            assert n == idx.numel() and torch.equal(aux["idx"][b, :n].long(), idx)
            if n:
                assert (aux["v"][b, :n].double() - v[b, idx]).norm() <= _bound(d, B) * v[b, idx].norm()
                h = (v * u)[b, idx]
                assert (aux["h"][b, :n].double() - h).norm() <= 2 * _bound(d, B) * h.norm()
    want = res.double() + (v * u) @ w[2].double()
    y = P.mlp_dense(layer, x, residual=res, ws=ws)
    assert ((y.double() - want).norm() / want.norm()).item() <= _bound(d, B)
    assert torch.equal(P.mlp_forward(layer, x, math.inf, residual=res, ws=ws), res)


@pytest.mark.parametrize("d,m,B", [(4096, 300, 8), (2856, 3000, 7), (1032, 3000, 16), (5128, 700, 4), (512, 5000, 8),
                                   (1024, 8000, 11)])
def test_batched_rmsnorm(d, m, B):
    P = _P()
    w, x, _ = _inputs(d, m, B, 3)
    x[B - 1] *= 1e-3  # a row whose own scale matters
    xn = x.double() / torch.sqrt((x.double() ** 2).mean(dim=1, keepdim=True) + EPS)
    g, u = (xn @ w[i].double().t() for i in range(2))
    t = _gap(_silu(g).abs(), 0.5)
    h = torch.where(_silu(g).abs() >= t, _silu(g) * u, torch.zeros_like(g))
    want = h @ w[2].double()
    y = P.stack_forward(P.Stack([P.Layer(*w)], [t]), x, eps=EPS).double() - x.double()
    # (the stream's own rounding, 2^-24 of x, on top)
    slack = 2.0 ** -23 * x.abs().max().item() * math.sqrt(d)
    for b in range(B):
        assert (y[b] - want[b]).norm() <= _bound(d, B) * want[b].norm() + slack


@pytest.mark.parametrize("d,m,B", [(1032, 3000, 8), (5128, 700, 4)])
def test_batched_special_values(d, m, B):
    """Three planes: an infinity or NaN in one row spoils that row alone, as it
    does in fp32 products."""
    P = _P()
    w, x, _ = _inputs(d, m, B, 11)
    x[1, 7] = float("inf")
    x[2, 9] = float("nan")
    y = P.mlp_dense(P.Layer(*w), x)
    x64 = x.double()
    want = (_silu(x64 @ w[0].double().t()) * (x64 @ w[1].double().t())) @ w[2].double()
    assert not torch.isfinite(y[1]).any() and torch.isnan(y[2]).all()
    for b in (0, *range(3, B)):
        assert (y[b].double() - want[b]).norm() <= _bound(d, B) * want[b].norm()


def _two_planes(x):
    hi = x.bfloat16().float()
    return hi.double() + (x - hi).bfloat16().double()


def _rel(a, b):
    return ((a.double() - b).norm() / b.norm()).item()


@pytest.mark.parametrize("d,m,B", [(1032, 3000, 8), (1032, 3000, 16), (5128, 700, 4)])
def test_batched_three_planes_of_x(d, m, B):
    """All 24 bits of x count, whatever its exponent: neighbouring channels of
    nearly equal values meet opposite weights, so a product is what the low
    bits differ by, and each pair is scaled by a power of two from 2^-60 to 2^60
    that its weights undo.  What is left of a term is 2^-12 of it; fp32 sums round
    2^-24 of a partial sum of some sqrt(d) terms, 2^-12 of the result a step and
    2^-10 in all; two planes round each x by 2^-19 (root mean square), 2^-7 of a
    gate or up result."""
    P = _P()
    g = torch.Generator(device="cuda").manual_seed(d + B)
    r = torch.rand((B, d // 2), generator=g, device="cuda") + 0.5
    x = torch.empty((B, d), device="cuda")
    x[:, 0::2] = r
    x[:, 1::2] = r - r * 2.0 ** -12 * (1 + torch.rand(r.shape, generator=g, device="cuda"))
    e = torch.randint(-60, 61, (d // 2,), generator=g, device="cuda").repeat_interleave(2).double()
    w = []
    for _ in range(2):
        half = (torch.randn((m, d // 2), generator=g, device="cuda") * 64).bfloat16()
        full = torch.empty((m, d), dtype=torch.bfloat16, device="cuda")
        full[:, 0::2], full[:, 1::2] = half, -half
        w.append((full.double() * 2.0 ** -e).bfloat16())
    w.append((torch.randn((m, d), generator=g, device="cuda") * 0.05).bfloat16())
    xs = (x.double() * 2.0 ** e).float()

    def ref(z):
        return (_silu(z @ w[0].double().t()) * (z @ w[1].double().t())) @ w[2].double()

    want = ref(xs.double())
    got, two = _rel(P.mlp_dense(P.Layer(*w), xs), want), _rel(ref(_two_planes(xs)), want)
    print(f"[planes] x {d}x{m} B{B}: {got:.2e}, two planes {two:.2e}")
    assert got <= 2.0 ** -10 and two >= 2.0 ** -7


@pytest.mark.parametrize("d,m,B", [(1032, 3000, 8), (1032, 3000, 16), (5128, 700, 4)])
def test_batched_three_planes_of_h(d, m, B):
    """All 24 bits of h count: pairs of neurons that differ in one weight of
    W_up, by about 2^-12 of their h, meet opposite rows of W_down.  An h carries
    some 2^-23 of its fp32 sums, 2^-11 of the difference; two planes would round
    it by 2^-19 (root mean square), 2^-7 of it."""
    P = _P()
    w, x, _ = _inputs(d, m, B, d + 2 * B)
    w = [v.clone() for v in w]
    for i in range(2):
        w[i][1::2] = w[i][0::2]
    w[1][0::2, 5], w[1][1::2, 5] = 0.0, 2.0 ** (-12 if d < 2048 else -11)
    w[2][1::2] = -w[2][0::2]
    x64 = x.double()
    h = _silu(x64 @ w[0].double().t()) * (x64 @ w[1].double().t())
    want = h @ w[2].double()
    two = _rel(_two_planes(h.float()) @ w[2].double(), want)
    got = _rel(P.mlp_dense(P.Layer(*w), x), want)
    print(f"[planes] h {d}x{m} B{B}: {got:.2e}, two planes {two:.2e}")
    assert got <= 2.0 ** -9 and two >= 2.0 ** -7


@pytest.mark.parametrize("d,m,B", [(1032, 3000, 8), (1032, 3000, 16), (5128, 700, 4)])
def test_batched_infinite_weights(d, m, B):
    """Three planes: an infinite weight makes of a result what it makes of it in
    fp32 products (its other planes are zero for many x and h, and 0 x inf is
    NaN): one in W_down leaves all other columns alone, one in W_up makes every
    column infinite, one in W_gate every column of the rows it turns positive."""
    P = _P()
    w, x, _ = _inputs(d, m, B, 17)
    x = torch.where(x.abs() < 0.1, torch.ones_like(x), x)  # no zeros; 1 has only its first plane
    x[:, 3] = torch.where(torch.arange(B, device="cuda") % 2 == 0, 1.0, -1.0)
    for which, j, c, sign in ((2, 5, 11, 1.0), (2, m - 1, d - 1, -1.0), (1, 5, 3, -1.0), (0, 5, 3, 1.0)):
        wi = [v.clone() for v in w]
        wi[which][j, c] = sign * math.inf
        wi[2][j] = torch.where(wi[2][j] == 0, torch.ones_like(wi[2][j]), wi[2][j])
        x64 = x.double()
        h = _silu(x64 @ wi[0].double().t()) * (x64 @ wi[1].double().t())
        want = h @ wi[2].double()
        inf = torch.isinf(want)
        assert inf.any() and (which == 0 or not torch.isnan(want).any())
        for y in (P.mlp_dense(P.Layer(*wi), x), P.mlp_forward(P.Layer(*wi), x, 0.0)):
            assert torch.equal(torch.isnan(y), torch.isnan(want))
            assert torch.equal(y[inf].double(), want[inf])
            for b in range(B):
                ok = torch.isfinite(want[b])
                if ok.any():
                    assert (y[b, ok].double() - want[b, ok]).norm() <= _bound(d, B) * want[b, ok].norm()
