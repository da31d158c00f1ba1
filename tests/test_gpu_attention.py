"""The library's causal attention by itself (il_test_attention) against float64 sums over the visible keys only."""
import numpy as np
import pytest

from paper_2010_04116_amd import binding as b

pytestmark = pytest.mark.gpu
IL = {"f32": b.IL_F32, "bf16": b.IL_BF16}


def reference(qkv, g, B, T, H, dh, stored_o=None):
    """float64: row q of the result is made of keys 0..q and of nothing else, so what is not finite in a token
    reaches exactly the rows that see it.  stored_o: the o whose row sums with g the backward takes."""
    d = H * dh
    x = qkv.astype(np.float64).reshape(B, T, 3, H, dh).transpose(2, 0, 3, 1, 4)
    q, k, v = x[0], x[1], x[2]
    go = g.astype(np.float64).reshape(B, T, H, dh).transpose(0, 2, 1, 3)
    sc = dh ** -0.5
    o = np.zeros((B, H, T, dh))
    so = None if stored_o is None else stored_o.astype(np.float64).reshape(B, T, H, dh).transpose(0, 2, 1, 3)
    dq, dk, dv = np.zeros_like(o), np.zeros_like(o), np.zeros_like(o)
    with np.errstate(all="ignore"):
        for t in range(T):
            s = np.einsum("bhi,bhui->bhu", q[:, :, t], k[:, :, :t + 1]) * sc
            m = np.where(np.isneginf(s.max(axis=2, keepdims=True)), 0, s.max(axis=2, keepdims=True))
            p = np.exp(s - m)
            p = p / p.sum(axis=2, keepdims=True)
            o[:, :, t] = np.einsum("bhu,bhui->bhi", p, v[:, :, :t + 1])
            D = ((o if so is None else so)[:, :, t] * go[:, :, t]).sum(axis=2, keepdims=True)
            ds = p * (np.einsum("bhi,bhui->bhu", go[:, :, t], v[:, :, :t + 1]) - D)
            dq[:, :, t] = np.einsum("bhu,bhui->bhi", ds, k[:, :, :t + 1]) * sc
            dk[:, :, :t + 1] += ds[..., None] * q[:, :, t][:, :, None] * sc
            dv[:, :, :t + 1] += p[..., None] * go[:, :, t][:, :, None]
    rows = lambda a: a.transpose(0, 2, 1, 3).reshape(B * T, d)  # noqa: E731
    return rows(o), np.concatenate([rows(dq), rows(dk), rows(dv)], axis=1)


def run(dtype, qkv, g, B, T, H, dh):
    import torch
    dev, tt = torch.device("cuda:0"), torch.float32 if dtype == "f32" else torch.bfloat16
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(tt).to(dev)  # noqa: E731
    d, N = H * dh, B * T
    dqkv_in, dg = to(qkv), to(g)
    o = torch.full((N, d), 7.0, dtype=tt, device=dev)
    lse = torch.full((B, H, T), 7.0, device=dev)
    out = torch.full((N, 3 * d), 7.0, dtype=tt, device=dev)
    dsum = torch.zeros(N * max(H, (d + 31) // 32), device=dev)
    args = (IL[dtype], dqkv_in, B, T, H, dh, o, lse)
    stream = torch.cuda.current_stream().cuda_stream
    if b.il_attention_wants_dsum(IL[dtype], dh):
        b.il_test_attention(*args, stream=stream)
        dsum = (dg.float() * o.float()).reshape(N, d // 32, 32).sum(dim=2).t().contiguous()
    b.il_test_attention(*args, dg, 1, out, dsum, stream=stream)
    torch.cuda.synchronize()
    return o.float().cpu().numpy(), out.float().cpu().numpy()


def bf16(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16).float().numpy()


def draw(seed, B, T, H, dh):
    rng = np.random.default_rng(seed)
    return bf16(rng.standard_normal((B * T, 3 * H * dh))), bf16(rng.standard_normal((B * T, H * dh)))


def held(got, want, dtype, what):
    """fp32 sums of a few hundred terms, and for bf16 one rounding to eight bits of the final value."""
    assert np.array_equal(np.isnan(got), np.isnan(want)), what + ": NaN in other places"
    fin = np.isfinite(want)
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)]), what
    scale = np.sqrt(np.mean(want[fin] ** 2)) if fin.any() else 1.0
    tol = 2e-5 * (scale + np.abs(want[fin])) + (2 ** -8 * np.abs(want[fin]) if dtype == "bf16" else 0)
    bad = np.abs(got[fin] - want[fin]) - tol
    assert bad.size == 0 or bad.max() <= 0, f"{what}: off by {np.abs(got[fin] - want[fin]).max():.3e}"


# nothing is rounded below the type of the inputs and outputs: neither probabilities nor their gradients
FP32_PRODUCTS = [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16), ("bf16", 32)]


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("T", [1, 17, 64, 150])
def test_forward_and_backward(dtype, dh, T):
    B, H = 2, 2
    qkv, g = draw(T, B, T, H, dh)
    print("case", dtype, dh, T, flush=True)
    o, dqkv = run(dtype, qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh, stored_o=o)
    held(o, wo, dtype, "o")
    held(dqkv, wd, dtype, "dqkv")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("T,token", [(17, 5), (64, 40), (90, 16), (90, 31), (90, 89)])
@pytest.mark.parametrize("part,value", [("q", np.nan), ("k", np.nan), ("v", np.nan), ("v", np.inf), ("g", np.nan), ("g", -np.inf)])
def test_what_is_not_finite_stays_with_the_rows_that_see_it(dtype, dh, T, token, part, value):
    B, H = 1, 2
    qkv, g = draw(T + token, B, T, H, dh)
    d = H * dh
    if part == "g":
        g[token, 3] = value
    else:
        qkv[token, {"q": 0, "k": d, "v": 2 * d}[part] + 3] = value
    print("case", dtype, dh, T, token, part, value, flush=True)
    o, dqkv = run(dtype, qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh)
    held(o, wo, dtype, "o")
    for i, what in enumerate(("dq", "dk", "dv")):
        got, want = dqkv[:, i * d:(i + 1) * d], wd[:, i * d:(i + 1) * d]
        assert np.array_equal(np.isfinite(got), np.isfinite(want)), what
        if dtype == "f32":
            held(np.where(np.isfinite(got), got, 0), np.where(np.isfinite(want), want, 0), dtype, what)


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("B,T", [(1, 15), (1, 16), (3, 33), (64, 64), (65, 64), (53, 150), (54, 150), (1, 511), (1, 512), (1, 530)])
def test_either_form_of_the_fp32_products(dtype, dh, B, T):
    """Both sides of the number of workgroups from which tiles are shared, and of the length from which narrow heads take
    eight wavefronts; the same bounds as above."""
    qkv, g = draw(B + T, B, T, 1, dh)
    print("case", dtype, dh, B, T, flush=True)
    o, dqkv = run(dtype, qkv, g, B, T, 1, dh)
    wo, wd = reference(qkv, g, B, T, 1, dh, stored_o=o)
    held(o, wo, dtype, "o")
    held(dqkv, wd, dtype, "dqkv")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("part,value", [("q", np.nan), ("k", np.nan), ("v", np.inf), ("g", -np.inf)])
def test_what_is_not_finite_where_tiles_are_shared(dtype, dh, part, value):
    B, T, H, token = 81, 90, 1, 64 * 90 + 31
    qkv, g = draw(7, B, T, H, dh)
    if part == "g":
        g[token, 3] = value
    else:
        qkv[token, {"q": 0, "k": dh, "v": 2 * dh}[part] + 3] = value
    print("case", dtype, dh, part, value, flush=True)
    o, dqkv = run(dtype, qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh)
    held(o, wo, dtype, "o")
    assert np.array_equal(np.isfinite(dqkv), np.isfinite(wd))
    if dtype == "f32":
        held(np.where(np.isfinite(dqkv), dqkv, 0), np.where(np.isfinite(wd), wd, 0), dtype, "dqkv")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("B,T,H,ns,split", [(18, 150, 3, 2, False), (12, 72, 7, 3, False), (5, 150, 3, 3, True), (1, 520, 2, 2, True)])
def test_streams_and_heads_in_either_form_of_the_fp32_products(dtype, dh, B, T, H, ns, split):
    """Several heads and stacked streams, each with gradients of its own; the same bounds as above."""
    import torch
    dev, tt = torch.device("cuda:0"), torch.float32 if dtype == "f32" else torch.bfloat16
    forms = b.il_attention_form(IL[dtype], dh, B, T, H), b.il_attention_form(IL[dtype], dh, B, T, H, ns)
    wide = 8 if dh <= 32 and T >= 512 else 4
    assert forms == ((wide, wide) if split else (0, 0)), forms
    d, N = H * dh, B * T
    qkv, _ = draw(B + T, B, T, H, dh)
    g = np.concatenate([draw(B + T + s, B, T, H, dh)[1] for s in range(1, ns + 1)])
    print("case streams", dtype, dh, B, T, H, ns, flush=True)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(tt).to(dev)  # noqa: E731
    o, lse = torch.full((N, d), 7.0, dtype=tt, device=dev), torch.full((B, H, T), 7.0, device=dev)
    out = torch.full((ns * N, 3 * d), 7.0, dtype=tt, device=dev)
    b.il_test_attention(IL[dtype], to(qkv), B, T, H, dh, o, lse, to(g), ns, out, torch.zeros(ns * N * max(H, (d + 31) // 32), device=dev),
                        stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    o, out = o.float().cpu().numpy(), out.float().cpu().numpy()
    for s in range(ns):
        wo, wd = reference(qkv, g[s * N:(s + 1) * N], B, T, H, dh, stored_o=o)
        held(out[s * N:(s + 1) * N], wd, dtype, f"dqkv of stream {s}")
    held(o, wo, dtype, "o")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("B,T,H,at,token", [(27, 90, 3, 20, 31), (1, 520, 2, 0, 131), (1, 520, 2, 0, 519)])
@pytest.mark.parametrize("part,value", [("q", np.nan), ("k", np.nan), ("v", np.inf), ("g", -np.inf)])
def test_what_is_not_finite_with_several_heads_and_long_rows(dtype, dh, B, T, H, at, token, part, value):
    """Tiles shared between the heads of a token, and rows that narrow heads divide over eight wavefronts."""
    want_form = 0 if B > 1 else 8 if dh <= 32 else 4
    assert b.il_attention_form(IL[dtype], dh, B, T, H) == b.il_attention_form(IL[dtype], dh, B, T, H, 1) == want_form
    qkv, g = draw(T, B, T, H, dh)
    d, row = H * dh, at * T + token
    if part == "g":
        g[row, dh + 3] = value
    else:
        qkv[row, {"q": 0, "k": d, "v": 2 * d}[part] + dh + 3] = value
    print("case", dtype, dh, B, T, H, token, part, value, flush=True)
    o, dqkv = run(dtype, qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh)
    held(o, wo, dtype, "o")
    assert np.array_equal(np.isfinite(dqkv), np.isfinite(wd))
    if dtype == "f32":
        held(np.where(np.isfinite(dqkv), dqkv, 0), np.where(np.isfinite(wd), wd, 0), dtype, "dqkv")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("B,T,H", [(27, 90, 3), (1, 520, 2)])
@pytest.mark.parametrize("low", [-1e31, -1e37, -np.inf])
def test_scores_below_any_mask_value_with_several_heads_and_long_rows(dtype, dh, B, T, H, low):
    """As test_scores_below_any_mask_value, with shared tiles and over eight wavefronts."""
    qkv, g = draw(3, B, T, H, dh)
    x = qkv.reshape(B, T, 3, H, dh)
    x[:, :, 0] = 0
    x[:, :, 0, :, 0] = 1e19
    x[:, :, 1] = 0
    if np.isinf(low):
        x[:, 1::2, 1, :, 0] = -3e38
    else:
        x[:, :, 1, :, 0] = low * dh ** 0.5 / 1e19
    t = np.arange(T)
    x[:, :, 2] = (t % 128)[None, :, None, None]          # (whole numbers that bf16 holds)
    print("case", dtype, dh, B, T, H, low, flush=True)
    o, _ = run(dtype, bf16(qkv), g, B, T, H, dh)
    seen = t % 2 == 0 if np.isinf(low) else t >= 0
    want = np.cumsum(t % 128 * seen) / np.cumsum(seen)
    held(o, np.tile(want[:, None], (B, H * dh)), dtype, "o")


@pytest.mark.parametrize("dtype,dh", FP32_PRODUCTS)
@pytest.mark.parametrize("low", [-1e31, -1e37, -np.inf])
def test_scores_below_any_mask_value(dtype, dh, low):
    """The first tokens' scores are all equal and lie far below -1e30; a later block's are -inf for every other key.
    Masked keys hold another value of V and must not show."""
    B, T, H = 1, 90, 2
    qkv, g = draw(3, B, T, H, dh)
    x = qkv.reshape(T, 3, H, dh)
    x[:, 0] = 0
    x[:, 0, :, 0] = 1e19                       # q . k = 1e19 k_0
    x[:, 1] = 0
    if np.isinf(low):
        x[1::2, 1, :, 0] = -3e38               # -inf in fp32: weighs nothing; the others score 0
    else:
        x[:, 1, :, 0] = low * dh ** 0.5 / 1e19
    x[:, 2] = np.arange(T)[:, None, None]
    qkv = bf16(qkv)
    print("case", dtype, dh, low, flush=True)
    o, _ = run(dtype, qkv, g, B, T, H, dh)
    t = np.arange(T)
    want = t / 2 if not np.isinf(low) else np.floor(t / 2)   # the mean of 0..t, of the even ones among them
    held(o, np.repeat(want[:, None], H * dh, axis=1), dtype, "o")


@pytest.mark.parametrize("dh,T,H", [(64, 64, 2), (64, 512, 2), (64, 513, 2), (64, 129, 130), (128, 100, 2), (128, 260, 1),
                                    (256, 64, 1), (256, 65, 1), (256, 256, 1), (256, 257, 1)])
def test_bf16_products(dh, T, H):
    """The bf16 matrix kernels at both sides of every line of their choice of workgroup.  Probabilities and dS are
    rounded to bf16, 2^-9 each at most and independently, as is the result: 2^-8 of the norm, and twice that for
    dQ, dK through two such factors."""
    B = 2 if H <= 2 else 1
    if H * dh > 2048:
        B, H = B * H // 13, 13                 # (many workgroups: several batches instead)
    qkv, g = draw(dh + T, B, T, H, dh)
    print("case bf16", dh, T, B, H, flush=True)
    o, dqkv = run("bf16", qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh, stored_o=o)
    assert np.linalg.norm(o - wo) <= 2 ** -8 * np.linalg.norm(wo)
    assert np.abs(o - wo).max() <= 2 ** -7 * np.abs(wo).max()
    for i in range(3):
        got, want = (a[:, i * H * dh:(i + 1) * H * dh] for a in (dqkv, wd))
        assert np.linalg.norm(got - want) <= 2 ** -7 * np.linalg.norm(want), "QKV"[i]
        rows = np.sqrt(((got - want) ** 2).sum(axis=1) / np.maximum((want ** 2).sum(axis=1), (want ** 2).sum() / len(want)))
        assert rows.max() <= 2 ** -5, ("QKV"[i], int(rows.argmax()))


@pytest.mark.parametrize("dh,B,T,H,ns", [
    (64, 1, 65, 1, 1), (64, 2, 300, 3, 2), (64, 8, 256, 8, 1), (64, 8, 257, 8, 1), (64, 16, 255, 2, 1), (64, 2, 416, 8, 1), (64, 2, 450, 8, 1),
    (128, 1, 65, 2, 2), (128, 2, 97, 16, 1), (128, 16, 257, 1, 1), (128, 1, 512, 16, 1), (128, 2, 1023, 4, 1),
    (256, 1, 2, 1, 1), (256, 1, 33, 2, 3), (256, 32, 64, 2, 1), (256, 33, 64, 2, 1), (256, 20, 64, 2, 1), (256, 1, 96, 8, 3), (256, 5, 128, 8, 1), (256, 7, 128, 8, 1), (256, 1, 512, 7, 2)])
def test_bf16_products_split_over_wavefronts(dh, B, T, H, ns):
    """About the lines from which a row's keys are divided up, several streams; the bounds of the test above."""
    print("case split", dh, B, T, H, ns, flush=True)
    bf16_against_float64(dh, B, T, H, ns)


# ragged lengths in grids that are large enough: the forward by four (0) and by two (-1) wavefronts, the backward (0) and
# its pairs of streams (-2); beside the line for width 128 also the split forward (4) with a shared backward
@pytest.mark.parametrize("dh,B,T,H,ns,forward,backward", [
    (64, 9, 200, 12, 1, -1, 0), (64, 40, 33, 8, 1, 0, 0), (64, 3, 600, 13, 1, 0, 0), (64, 40, 129, 8, 2, 0, -2),
    (128, 9, 100, 8, 1, 0, 0), (128, 5, 257, 8, 2, 0, 0), (128, 9, 33, 8, 3, 0, 0), (128, 3, 1000, 6, 1, 0, 0), (128, 1, 600, 14, 1, 0, 0),
    (128, 1, 513, 5, 3, 4, 0),
    (256, 9, 97, 8, 1, -1, 0), (256, 9, 257, 4, 2, 0, 0), (256, 17, 513, 2, 1, 0, 0), (256, 70, 31, 4, 3, 0, 0), (256, 40, 130, 8, 1, 0, 0)])
def test_bf16_products_with_shared_tiles(dh, B, T, H, ns, forward, backward):
    """What larger grids take, at lengths that no tile divides; the bounds of the tests above."""
    print("case shared", dh, B, T, H, ns, flush=True)
    assert (b.il_attention_form(b.IL_BF16, dh, B, T, H), b.il_attention_form(b.IL_BF16, dh, B, T, H, ns)) == (forward, backward)
    bf16_against_float64(dh, B, T, H, ns)


def bf16_against_float64(dh, B, T, H, ns):
    import torch
    dev, d, N = torch.device("cuda:0"), H * dh, B * T
    gen = torch.Generator(device=dev).manual_seed(dh + T)
    qkv = torch.randn(N, 3 * d, generator=gen, device=dev).to(torch.bfloat16)
    g = torch.randn(ns * N, d, generator=gen, device=dev).to(torch.bfloat16)
    o, lse = torch.full((N, d), 7.0, dtype=torch.bfloat16, device=dev), torch.full((B, H, T), 7.0, device=dev)
    out = torch.full((ns * N, 3 * d), 7.0, dtype=torch.bfloat16, device=dev)
    stream = torch.cuda.current_stream().cuda_stream
    b.il_test_attention(b.IL_BF16, qkv, B, T, H, dh, o, lse, stream=stream)
    dsum = (g.float().reshape(ns, N, d) * o.float()).reshape(ns * N, d // 32, 32).sum(dim=2).t().contiguous()
    b.il_test_attention(b.IL_BF16, qkv, B, T, H, dh, o, lse, g, ns, out, dsum, stream=stream)
    q, k, v = (x.reshape(B, T, H, dh).transpose(1, 2).float().contiguous() for x in qkv.reshape(N, 3, d).unbind(1))
    S = (q.double() @ k.double().transpose(2, 3).contiguous()) * dh ** -0.5
    S = S.masked_fill(torch.ones(T, T, dtype=torch.bool, device=dev).triu(1), float("-inf"))
    P = torch.softmax(S, dim=3)
    rows = lambda a: a.transpose(1, 2).reshape(N, d)  # noqa: E731

    def near(got, want, tol, what):
        got = got.double()
        assert (got - want).norm() <= tol * want.norm(), what
        assert (got - want).abs().max() <= 2 * tol * want.abs().max(), what
        e = (got - want).square().sum(1) / want.square().sum(1).clamp_min(want.square().sum() / len(want))
        assert e.max().sqrt() <= 4 * tol, (what, int(e.argmax()))

    near(o, rows(P @ v.double()), 2 ** -8, "o")
    got_lse, want_lse = lse.double() / np.log2(np.e), torch.logsumexp(S, dim=3)    # (powers of two)
    assert (got_lse - want_lse).abs().max() <= 1e-5 * want_lse.abs().max()
    for s in range(ns):
        go = g[s * N:(s + 1) * N].reshape(B, T, H, dh).transpose(1, 2).double().contiguous()
        D = (go * o.reshape(B, T, H, dh).transpose(1, 2).double()).sum(3, keepdim=True)
        dS = P * (go @ v.double().transpose(2, 3).contiguous() - D) * dh ** -0.5
        want = (dS @ k.double(), dS.transpose(2, 3).contiguous() @ q.double(), P.transpose(2, 3).contiguous() @ go)
        for i in range(3):
            near(out[s * N:(s + 1) * N, i * d:(i + 1) * d], rows(want[i]), 2 ** -7, (s, "QKV"[i]))


@pytest.mark.parametrize("dh", [64, 128, 256])
@pytest.mark.parametrize("part,value", [("q", np.nan), ("k", np.nan), ("v", np.nan), ("v", np.inf), ("g", np.nan), ("g", -np.inf)])
def test_what_is_not_finite_where_bf16_products_are_split(dh, part, value):
    """It reaches the rows that see it.  Rows of other 32-row blocks that do not are as they were; in its own block a
    masked weight of zero meets it in a product, so nothing is asked of the rows there that do not see it."""
    B, T, H, token = 1, 200, 2, 70
    lo, hi = token // 32 * 32, token // 32 * 32 + 32
    qkv, g = draw(dh, B, T, H, dh)
    d = H * dh
    clean = run("bf16", qkv, g, B, T, H, dh)
    if part == "g":
        g[token, 3] = value
    else:
        qkv[token, {"q": 0, "k": d, "v": 2 * d}[part] + 3] = value
    print("case bf16 not finite", dh, part, value, flush=True)
    form = b.il_attention_form(b.IL_BF16, dh, B, T, H)
    assert form == b.il_attention_form(b.IL_BF16, dh, B, T, H, 1) == (2 if dh == 256 else 4)
    o, dqkv = run("bf16", qkv, g, B, T, H, dh)
    wo, wd = reference(qkv, g, B, T, H, dh)
    rows = np.arange(T)
    by_query, by_key = (rows < lo) | (rows >= token), (rows <= token) | (rows >= hi)
    for got, want, was, asked, what in [(o, wo, clean[0], by_query, "o"), (dqkv[:, :d], wd[:, :d], clean[1][:, :d], by_query, "dq"),
                                        (dqkv[:, d:2 * d], wd[:, d:2 * d], clean[1][:, d:2 * d], by_key, "dk"),
                                        (dqkv[:, 2 * d:], wd[:, 2 * d:], clean[1][:, 2 * d:], by_key, "dv")]:
        assert np.array_equal(np.isfinite(got)[asked], np.isfinite(want)[asked]), what
        same = asked & ((rows < token) if what in ("o", "dq") else (rows > token))   # never meets the token
        assert np.array_equal(got[same & np.isfinite(want).all(axis=1)], was[same & np.isfinite(want).all(axis=1)]), what


@pytest.mark.parametrize("dh,B,T,H,ns", [
    (64, 5, 256, 16, 2), (64, 5, 256, 16, 3), (64, 10, 129, 16, 2), (64, 5, 1000, 8, 2), (64, 40, 33, 8, 2), (64, 160, 1, 2, 3),
    (64, 27, 64, 4, 5), (64, 1, 64, 1, 2), (128, 4, 200, 11, 2), (256, 8, 65, 4, 3)])
def test_streams_that_share_a_walk(dh, B, T, H, ns):
    """Streams taken together give what each gives by itself, bit for bit: the same products and sums in the same order.
    Both sides of the number of workgroups from which streams go in pairs, even and odd numbers of them."""
    import torch
    dev, d, N = torch.device("cuda:0"), H * dh, B * T
    print("case streams", dh, B, T, H, ns, flush=True)
    gen = torch.Generator().manual_seed(dh + T)
    qkv = torch.randn(N, 3 * d, generator=gen).to(torch.bfloat16).to(dev)
    g = torch.randn(ns * N, d, generator=gen).to(torch.bfloat16).to(dev)
    g[(ns - 1) * N + N // 2, 0] = float("nan")   # one stream's alone
    o, lse = torch.empty(N, d, dtype=torch.bfloat16, device=dev), torch.empty(B, H, T, device=dev)
    stream = torch.cuda.current_stream().cuda_stream
    b.il_test_attention(b.IL_BF16, qkv, B, T, H, dh, o, lse, stream=stream)

    def backward(g, streams):
        dsum = (g.float().reshape(streams, N, d) * o.float()).reshape(streams * N, d // 32, 32).sum(dim=2).t().contiguous()
        out = torch.full((streams * N, 3 * d), 7.0, dtype=torch.bfloat16, device=dev)
        b.il_test_attention(b.IL_BF16, qkv, B, T, H, dh, o, lse, g, streams, out, dsum, stream=stream)
        return out

    out = backward(g, ns)
    for s in range(ns):
        one = backward(g[s * N:(s + 1) * N].contiguous(), 1)
        assert torch.equal(one.isnan(), out[s * N:(s + 1) * N].isnan()) and bool(one.isnan().any()) == (s == ns - 1), s
        assert torch.equal(one.nan_to_num(), out[s * N:(s + 1) * N].nan_to_num()), s
