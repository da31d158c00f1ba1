"""LayerNorm's kernels by themselves, through the C ABI's test hooks."""
import numpy as np
import pytest

from paper_2010_04116_amd import binding as b

pytestmark = pytest.mark.gpu


def _row_sum(x, V):
    """A wavefront's sum of each row: a lane adds its columns (lane + 64 j) V + e in order, lanes then meet pairwise."""
    rows, d = x.shape
    J = -(-d // (64 * V))
    p = np.zeros((rows, 64 * V * J), np.float32)
    p[:, :d] = x
    lanes = p.reshape(rows, J, 64, V).transpose(0, 2, 1, 3).reshape(rows, 64, J * V)
    s = np.zeros((rows, 64), np.float32)
    for i in range(J * V):
        s += lanes[:, :, i]
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[:, np.arange(64) ^ o]
    return s[:, 0]


@pytest.mark.parametrize("dtype,widths", [("f32", (64, 320, 768, 1024, 2048, 250, 1001)), ("bf16", (64, 320, 768, 1024, 1280, 1536, 2048))])
@pytest.mark.parametrize("offset", [0.0, 5.0, 1000.0])
def test_forward_centres_a_row_in_one_rounding(dtype, widths, offset):
    """y = fl(x - S / d) * rstd with the fp32 sum S: x minus S times fl(1 / d), rounded once, and the same value for the
    variance and for y (gain 1, bias 0).  A mean that is rounded first changes y wherever 1 / d is not exact, and by
    more the larger the mean is (in bf16 from an offset of some hundreds on).  One element in 10^4 may differ by a last
    bit: float64 holds S * fl(1 / d) exactly but rounds the difference once more."""
    import torch
    rows, eps = 37, 1e-5
    tt, code = (torch.float32, b.IL_F32) if dtype == "f32" else (torch.bfloat16, b.IL_BF16)
    for d in widths:
        rng = np.random.default_rng(d)
        x = (rng.normal(size=(rows, d)) + offset).astype(np.float32)
        gain = lambda v: torch.full((d,), v, device="cuda:0", dtype=tt)  # noqa: E731
        y, stats = torch.empty(rows, d, device="cuda:0", dtype=tt), torch.empty(rows, 2, device="cuda:0")
        copy = torch.empty(rows, d, device="cuda:0")
        print("case layernorm", dtype, d, offset, flush=True)
        b.il_test_layernorm(code, torch.from_numpy(x).to("cuda:0"), gain(1.0), gain(0.0), eps, rows, d, y, stats, copy,
                            stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        y, stats = y.float().cpu().numpy(), stats.cpu().numpy()
        S, inv = _row_sum(x, 4 if d % 4 == 0 else 1).astype(np.float64), np.float64(np.float32(1) / np.float32(d))
        centred = (x.astype(np.float64) - (S * inv)[:, None]).astype(np.float32)
        want = torch.from_numpy(centred * stats[:, 1:]).to(tt).float().numpy()
        assert np.array_equal(copy.cpu().numpy(), x) and np.array_equal(stats[:, 0], (S * inv).astype(np.float32))
        assert np.count_nonzero(y != want) <= 1e-4 * y.size, (d, np.count_nonzero(y != want) / y.size)
        assert np.all(np.abs(y - want) <= 2.0 ** (-23 if dtype == "f32" else -7) * np.abs(want)), d
        rstd = 1 / np.sqrt((centred.astype(np.float64) ** 2).sum(axis=1) * inv + eps)
        # a sum of squares of d / 64 additions in a lane and six across, then the hardware's reciprocal root
        assert np.all(np.abs(stats[:, 1] / rstd - 1) <= (d / 64 + 12) * 2.0 ** -24), d


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("weights", [(1.0,), (0.5,), (1.0, 1.0), (0.0, 1.0), (0.5, 0.0, 0.5), (1.0, 1.0, 0.0, 1.0, 1.0)])
@pytest.mark.parametrize("tokens,d", [(1, 260), (3, 512), (65, 512), (130, 516), (515, 768), (7, 1024), (1030, 1024), (33, 1028), (520, 2048)])
def test_backward_leaves_the_sum_of_the_streams(dtype, weights, tokens, d):
    """The form that leaves the streams' sum changes nothing else - G, Gb and the gain's and bias's gradients are those
    of the form that does not, bit for bit or to the order of fp32 sums - and the sum is that of the stored streams: fp32
    products added in order, rounded once; its column sums are taken before that rounding.  A stream of weight zero may
    hold anything."""
    import torch
    ns, code = len(weights), b.IL_F32 if dtype == "f32" else b.IL_BF16
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    print("case layernorm backward", dtype, weights, tokens, d, flush=True)
    gen = torch.Generator().manual_seed(tokens + d + ns)
    rnd = lambda *s: torch.randn(*s, generator=gen).to("cuda:0")  # noqa: E731
    dy, x, gamma, G0 = rnd(ns * tokens, d).to(tt), rnd(tokens, d) + 1.0, (1 + 0.1 * rnd(d)).to(tt), rnd(ns * tokens, d)
    idle = [s for s, w in enumerate(weights) if w == 0.0]
    for s in idle:
        G0[s * tokens + tokens // 2, d // 2] = float("nan")
    stats = torch.stack([x.mean(1), (x.var(1, unbiased=False) + 1e-5).rsqrt()], 1).contiguous()
    out = []
    for summed in (False, True):
        G, Gb = G0.clone(), torch.full((ns * tokens, d), 7.0, dtype=tt, device="cuda:0")
        part, ypart = torch.full((512, 2 * d), 7.0, device="cuda:0"), torch.full((512, d), 7.0, device="cuda:0")
        ysum = torch.full((tokens, d), 7.0, dtype=tt, device="cuda:0")
        blocks, made = b.il_test_layernorm_backward(code, dy, x, stats, gamma, ns, tokens, d, G, Gb, weights, part, ysum,
                                                    ypart if summed else None, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert made == summed and 1 <= blocks <= 512
        assert torch.all(part[blocks:] == 7.0) and torch.all(ypart[blocks if summed else 0:] == 7.0)
        out.append((G, Gb, part[:blocks].double().sum(0), ypart[:blocks].double().sum(0), ysum))
    (G, Gb, cols, _, untouched), (G2, Gb2, cols2, ycols, ysum) = out
    assert torch.all(untouched == 7.0)
    same = lambda p, q: torch.equal(p.nan_to_num(), q.nan_to_num()) and torch.equal(p.isnan(), q.isnan())  # noqa: E731
    assert same(G, G2) and same(Gb, Gb2) and same(Gb.float(), G.to(tt).float())
    live = [s for s, w in enumerate(weights) if w != 0.0]
    # against float64: the gradient at x, and the two column sums
    xd, dyd, gd = x.double(), dy.double().view(ns, tokens, d), gamma.double()
    xh = (xd - stats[:, :1].double()) * stats[:, 1:].double()
    dxh = dyd * gd
    want = G0.double().view(ns, tokens, d) + stats[:, 1:].double() * (
        dxh - dxh.mean(2, keepdim=True) - xh * (dxh * xh).mean(2, keepdim=True))
    for s in live:   # fp32: sums of d products (their roundings on the scale of the largest row), some ten operations beside
        err = (G.view(ns, tokens, d)[s].double() - want[s]).abs()
        assert float((err / (1 + want[s].abs() + stats[:, 1:].double() * (1 + xh.abs()))).max()) <= 40 * 2.0 ** -24
    w = torch.tensor(weights, dtype=torch.float64, device="cuda:0")[:, None, None]
    for c, terms in ((cols, w * dyd * xh), (cols2, w * dyd * xh)):
        n = terms.shape[0] * tokens
        bound = (n + 8) * 2.0 ** -24 * terms.abs().sum((0, 1)) + 1e-30
        assert bool(torch.all((c[:d] - terms.sum((0, 1))).abs() <= bound))
        assert bool(torch.all((c[d:] - (w * dyd).sum((0, 1))).abs() <= (n + 8) * 2.0 ** -24 * (w * dyd).abs().sum((0, 1)) + 1e-30))
    y = torch.zeros(tokens, d, device="cuda:0")
    for s in live:   # weights are powers of two: a product is exact
        y = y + weights[s] * Gb.view(ns, tokens, d)[s].float()
    assert torch.equal(ysum, y.to(tt))
    assert bool(torch.all((ycols - y.double().sum(0)).abs() <= (tokens + 8) * 2.0 ** -24 * y.double().abs().sum(0) + 1e-30))
