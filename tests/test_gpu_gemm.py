"""Kernel-level parity of the bf16 MFMA GEMM (every tile configuration, operand layout and
epilogue the step uses, ragged edges, segmented weight-gradient reduction) against a float64
matrix product of the same bf16-rounded operands.  Through the C ABI's il_test_gemm hook."""
import numpy as np
import pytest

from oracle import interlock as O
from paper_2010_04116_amd import binding as b, synth

pytestmark = pytest.mark.gpu
TILES = [1, 2, 3, 4, 5, 6, 7, 8]
# the (layout, epilogue) pairs the library instantiates: forward, data gradient, weight gradient
# (epilogue 7: the head's logits tile, stored as IEEE half)
_COMBOS = [(0, 1, 0), (0, 1, 1), (0, 1, 2), (0, 1, 3), (0, 0, 0), (0, 0, 4), (0, 0, 5), (1, 1, 6), (0, 1, 7)]


def _bf16(a):
    return synth.round_to_bf16(a.astype(np.float32))


_gelu, _gelu_grad = O.gelu, O.gelu_grad      # the oracle's tanh-GELU (pinned in test_oracle_primitives.py)


def run_case(M, N, K, akm, bkm, epi, tile, seed=0, beta=0, scale=1.0):
    import torch
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(seed)
    A = _bf16(rng.standard_normal((M, K)) * 0.5)
    B = _bf16(rng.standard_normal((K, N)) * 0.5)
    bias = _bf16(rng.standard_normal(N) * 0.5)
    res = rng.standard_normal((M, N)).astype(np.float32)
    aux_rows = max(1, M // 2)
    aux = _bf16(rng.standard_normal((aux_rows, N)))
    c0 = rng.standard_normal((M, N)).astype(np.float32)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    tb = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16).to(dev)
    tf = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    dA = tb(A.T if akm else A)
    dB = tb(B if bkm else B.T)
    f32out = epi in (3, 5, 6)
    C = tf(c0) if f32out else torch.zeros((M, N), dtype=torch.bfloat16, device=dev)
    C2 = torch.zeros((M, N), dtype=torch.bfloat16, device=dev)
    b.il_test_gemm(b.IL_BF16, dA, dB, M, N, K, M if akm else K, N if bkm else K, akm, bkm, epi, C, C2=C2,
                   ldc=N, bias=tb(bias), res=tf(res), aux=tb(aux), aux_wrap=aux_rows, scale=scale, beta=beta,
                   tile=tile, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = (C.view(torch.float16) if epi == 7 else C).float().cpu().numpy().astype(np.float64)
    if epi == 0:
        want = acc
    elif epi == 1:
        want = acc + bias
    elif epi == 2:
        want = acc + bias
        got2 = C2.float().cpu().numpy().astype(np.float64)
        want2 = _gelu(_bf16(want).astype(np.float64))
        assert np.linalg.norm(got2 - want2) <= 6e-3 * np.linalg.norm(want2)
    elif epi == 3:
        want = acc + bias + res
    elif epi == 4:
        want = acc * _gelu_grad(aux.astype(np.float64))[np.arange(M) % aux_rows]
    elif epi in (5, 7):
        want = acc
    else:
        want = scale * acc + (c0 if beta else 0)
    tol = 1e-5 if f32out else (8e-4 if epi == 7 else 6e-3)   # fp32 outputs: accumulation order only; bf16 / half: one rounding
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert err <= tol, f"M={M} N={N} K={K} akm={akm} bkm={bkm} epi={epi} tile={tile}: rel err {err:.3e}"
    if not f32out:
        assert np.max(np.abs(got - want)) <= (2 ** -10 if epi == 7 else 2 ** -7) * np.max(np.abs(want)) + 1e-6
    # no row, column or tile may hide inside the norm: every row and column to twice the tolerance
    # (on the scale of the RMS row / column for the nearly empty ones), every element to a bf16
    # rounding step of the largest value
    d2 = (got - want) ** 2
    for axis in (0, 1):
        nref = np.sqrt((want ** 2).sum(axis=axis))
        e = np.sqrt(d2.sum(axis=axis)) / np.maximum(nref, np.sqrt((nref ** 2).mean()))
        assert e.max() <= 2 * tol, f"M={M} N={N} K={K} epi={epi} tile={tile}: axis {axis} index {int(e.argmax())} rel err {e.max():.3e}"
    assert np.max(np.abs(got - want)) <= (1e-4 if f32out else 2 ** -7) * np.max(np.abs(want)) + 1e-6


@pytest.mark.parametrize("tile", TILES)
def test_forward_layout_all_epilogues(tile):
    for epi in (0, 1, 2, 3):
        run_case(384, 264, 192, 0, 1, epi, tile, seed=epi)


@pytest.mark.parametrize("tile", TILES)
def test_dgrad_layout_all_epilogues(tile):
    for epi in (0, 4, 5):
        run_case(520, 136, 320, 0, 0, epi, tile, seed=10 + epi)


@pytest.mark.parametrize("tile", TILES)
def test_wgrad_layout(tile):
    run_case(200, 392, 256, 1, 1, 6, tile, seed=20, beta=0, scale=0.5)
    run_case(200, 392, 256, 1, 1, 6, tile, seed=21, beta=1, scale=1.0)


@pytest.mark.parametrize("tile", TILES)
def test_k_tail_and_tiny_sizes(tile):
    run_case(8, 8, 8, 0, 0, 0, tile, seed=30)
    run_case(72, 40, 104, 0, 1, 1, tile, seed=31)      # K not a multiple of 32 or 64
    run_case(72, 40, 104, 0, 0, 5, tile, seed=32)
    run_case(40, 72, 72, 1, 1, 6, tile, seed=33)


@pytest.mark.parametrize("tile", [0] + TILES)
def test_multi_tile_shapes(tile):
    run_case(1024, 768, 512, 0, 1, 1, tile, seed=40)
    run_case(1024, 768, 512, 0, 0, 0, tile, seed=41)
    run_case(512, 1024, 2048, 1, 1, 6, tile, seed=42)


@pytest.mark.parametrize("tile,edge", [(1, 256), (3, 128), (5, 64)])
@pytest.mark.parametrize("tiles", [1, 7, 8, 9, 11, 23])
def test_tile_counts_on_either_side_of_eight(tiles, tile, edge):
    """Workgroups are dealt out over eight XCDs: every tile is taken once whatever the remainder."""
    run_case(edge * tiles - 8, 40, 64, 0, 1, 1, tile, seed=50 + tiles)
    run_case(edge + 8, edge * tiles, 64, 0, 0, 0, tile, seed=60 + tiles)


@pytest.mark.parametrize("M,N,tile", [(1768, 296, 5), (1768, 296, 4), (2104, 136, 3), (8200, 520, 1), (8264, 520, 7), (2104, 296, 6)])
def test_tall_outputs_whose_tiles_eight_does_not_divide(M, N, tile):
    """Their tiles are dealt in launch order: every one is taken once."""
    edge = {1: (256, 256), 3: (128, 128), 4: (64, 64), 5: (64, 64), 6: (256, 128), 7: (128, 256)}[tile]
    tm, tn = -(-M // edge[0]), -(-N // edge[1])
    assert tm * tn % 8 and b.il_gemm_tile_of(tm, tn, *edge, 1024, 9) == (1, 1)
    run_case(M, N, 1024, 0, 1, 1, tile, seed=60)
    run_case(M, N, 1024, 1, 1, 6, tile, seed=61, beta=1)


def test_library_choice_at_the_benchmark_shapes():
    """tile = 0 at output shapes of the benchmark workloads, one per branch of the tile choice
    (256x256; 128x128 four-stage; 128x256 / 256x128; 128x128 two-stage; 64x64 four-stage; 64x64),
    with a short K so that the float64 product stays cheap."""
    run_case(4096, 4096, 192, 0, 1, 2, 0, seed=50)      # 256 tiles of 256x256
    run_case(4096, 1024, 192, 0, 1, 3, 0, seed=51)      # 256 tiles of 128x128
    run_case(8192, 1024, 192, 0, 0, 0, 0, seed=52)      # 256 tiles of 128x256
    run_case(1024, 8192, 192, 1, 1, 6, 0, seed=53)      # 256 tiles of 256x128 (k-major operands)
    run_case(4096, 1536, 192, 0, 0, 5, 0, seed=54)      # 384 tiles of 128x128
    run_case(2048, 512, 192, 0, 1, 3, 0, seed=55)       # 256 tiles of 64x64
    run_case(2048, 1536, 192, 0, 1, 1, 0, seed=56)      # 768 tiles of 64x64


@pytest.mark.parametrize("tile", [0, 8])
def test_persistent_kernel_second_round_ragged(tile):
    """More than 256 tiles of 256x256 with ragged M and N (18 x 17 = 306 tiles), more than the chip has CUs: a
    second, partial round of workgroups.  Every (layout, epilogue) the step uses."""
    for i, (akm, bkm, epi) in enumerate(_COMBOS):
        M, N = (4360, 4104) if not akm else (4360 - 8, 4104)
        run_case(M, N, 128, akm, bkm, epi, tile, seed=70 + i, beta=int(epi == 6))


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 6, 7, 8])
def test_logits_epilogue_statistics(tile):
    """The head's logits GEMM leaves, beside the half-precision tile, the softmax statistics of every
    64-column group taken from its fp32 accumulators, and each row's target logit: checked against the
    float64 product (ragged M and N, a last group of 40 columns, targets at both ends and out of range)."""
    import torch
    dev = torch.device("cuda:0")
    for M, N, K, seed in ((300, 1000, 192, 90), (520, 4104, 128, 91)):
        rng = np.random.default_rng(seed)
        A = _bf16(rng.standard_normal((M, K)))
        B = _bf16(rng.standard_normal((K, N)) * 0.7)
        acc = A.astype(np.float64) @ B.astype(np.float64)
        tgt = rng.integers(0, N, size=M).astype(np.int32)
        tgt[:4] = [0, N - 1, -1, N]                      # edges, and two ignored positions
        G = (N + 63) // 64
        dA = torch.from_numpy(A).to(torch.bfloat16).to(dev)
        dB = torch.from_numpy(B).to(torch.bfloat16).to(dev)
        C = torch.zeros((M, N), dtype=torch.bfloat16, device=dev)
        S = torch.full((M * G * 2 + M,), -7.0, dtype=torch.float32, device=dev)
        b.il_test_gemm(b.IL_BF16, dA, dB, M, N, K, K, N, 0, 1, 7, C, C2=S, aux=torch.from_numpy(tgt).to(dev), tile=tile,
                       stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        z = C.view(torch.float16).float().cpu().numpy().astype(np.float64)
        assert np.abs(z - acc).max() <= 2 ** -10 * np.abs(acc).max() + 1e-6
        s = S.cpu().numpy().astype(np.float64)
        st, zt = s[:M * G * 2].reshape(M, G, 2), s[M * G * 2:]
        pad = np.full((M, G * 64), -np.inf)
        pad[:, :N] = acc
        grp = pad.reshape(M, G, 64)
        m = grp.max(axis=2)
        se = np.exp(grp - m[:, :, None]).sum(axis=2)
        assert np.abs(st[:, :, 0] - m).max() <= 1e-5 * np.abs(acc).max(), (M, N, tile)
        assert np.abs(st[:, :, 1] / se - 1).max() <= 2e-5, (M, N, tile)
        lse = np.log((st[:, :, 1] * np.exp(st[:, :, 0] - st[:, :, 0].max(axis=1, keepdims=True))).sum(axis=1)) \
            + st[:, :, 0].max(axis=1)
        ref = np.log(np.exp(acc - acc.max(axis=1, keepdims=True)).sum(axis=1)) + acc.max(axis=1)
        assert np.abs(lse - ref).max() <= 2e-5, (M, N, tile)
        ok = (tgt >= 0) & (tgt < N)
        want = acc[np.arange(M)[ok], tgt[ok]]
        assert np.abs(zt[ok] - want).max() <= 1e-5 * np.abs(acc).max(), (M, N, tile)
        assert np.all(zt[~ok] == -7.0)                       # ignored rows are left alone


def test_unsupported_combinations_are_rejected():
    import torch
    dev = torch.device("cuda:0")
    x = torch.zeros((64, 64), dtype=torch.bfloat16, device=dev)
    with pytest.raises(b.InterlockError) as e:       # k-major A with k-contiguous B is not a layout the step uses
        b.il_test_gemm(b.IL_BF16, x, x, 64, 64, 64, 64, 64, 1, 0, 0, x)
    assert e.value.status == b.IL_E_SHAPE
    with pytest.raises(b.InterlockError):            # N not a multiple of 8
        b.il_test_gemm(b.IL_BF16, x, x, 64, 60, 64, 64, 64, 0, 0, 0, x, ldc=64)
    with pytest.raises(b.InterlockError) as e:       # the logits epilogue has no 64x64 tile (32-wide wave tiles)
        b.il_test_gemm(b.IL_BF16, x, x, 64, 64, 64, 64, 64, 0, 1, 7, x, tile=4)
    assert e.value.status == b.IL_E_SHAPE




def test_seeded_random_shapes_every_tile_choice():
    """A seeded sweep over sizes from a single 8-wide sliver to several tiles with ragged edges in
    all three dimensions; tile = 0 lets the library choose, the others force each configuration."""
    rng = np.random.default_rng(20100411)
    dims = [8, 16, 24, 40, 64, 72, 120, 128, 136, 200, 256, 264, 328, 520]
    for case in range(45):
        M, N, K = (int(rng.choice(dims)) for _ in range(3))
        akm, bkm, epi = _COMBOS[case % len(_COMBOS)]
        tile = [0, 1, 2, 3, 4, 5, 6, 7, 0][case % 9]
        print("case", case, M, N, K, akm, bkm, epi, "tile", tile, flush=True)
        run_case(M, N, K, akm, bkm, epi, tile, seed=1000 + case, beta=case & 1, scale=0.5 if case & 2 else 1.0)


def test_long_reduction_and_thin_outputs():
    """The shapes of the head's data gradient (tiny output, very long K) and of a bias-sized sliver."""
    run_case(64, 8, 8192, 0, 0, 5, 0, seed=77)
    run_case(8, 64, 4104, 1, 1, 6, 0, seed=78, beta=1, scale=0.25)
    run_case(72, 8, 520, 0, 1, 3, 0, seed=79)


# fp32: tile edges and remainders in every direction, both load widths (16-byte rows or not), the tile the library
# chooses (the last shape fills the chip twice with 128x128 tiles), one K step and many
@pytest.mark.parametrize("M,N,K", [(64, 64, 32), (1, 3, 5), (65, 68, 36), (67, 129, 33), (128, 200, 260),
                                   (2816, 3000, 100)])
@pytest.mark.parametrize("akm,bkm", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_f32_gemm(M, N, K, akm, bkm):
    import torch
    rng = np.random.default_rng(M + 7 * N + K)
    x, y = (rng.normal(size=s).astype(np.float32) for s in ((M, K), (K, N)))
    res, bias = rng.normal(size=(M, N)).astype(np.float32), rng.normal(size=N).astype(np.float32)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")
    A, B = dev(x.T if akm else x), dev(y if bkm else y.T)
    C = torch.full((M, N), float("nan"), device="cuda:0")
    print("case f32", M, N, K, akm, bkm, flush=True)
    b.il_test_gemm(0, A, B, M, N, K, A.shape[1], B.shape[1], akm, bkm, 3, C, bias=dev(bias), res=dev(res))
    torch.cuda.synchronize()
    want = x.astype(np.float64) @ y + bias + res
    # K fused multiply-adds and two adds, each within 2^-24 of the running magnitude
    bound = (K + 2) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(y) + np.abs(bias) + np.abs(res))
    assert np.all(np.abs(C.cpu().numpy() - want) <= bound)


@pytest.mark.parametrize("tile", [2, 3, 4])
@pytest.mark.parametrize("akm,bkm,epi", [(0, 1, 3), (0, 0, 0), (1, 1, 6)])
@pytest.mark.parametrize("M,N,K", [(64, 64, 16), (128, 64, 64), (132, 68, 100), (260, 196, 292), (4, 4, 4)])
def test_f32_tiles(M, N, K, akm, bkm, epi, tile):
    """Each fp32 tile at its edges, with one K step, a part of one and several; values over twelve decades."""
    import torch
    rng = np.random.default_rng(M + 7 * N + K + tile)
    x, y = ((rng.normal(size=s) * 10.0 ** rng.uniform(-6, 6, size=s)).astype(np.float32) for s in ((M, K), (K, N)))
    res, bias = rng.normal(size=(M, N)).astype(np.float32), rng.normal(size=N).astype(np.float32)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")  # noqa: E731
    A, B = dev(x.T if akm else x), dev(y if bkm else y.T)
    C = torch.full((M, N), float("nan"), device="cuda:0")
    print("case f32", M, N, K, akm, bkm, epi, tile, flush=True)
    b.il_test_gemm(0, A, B, M, N, K, A.shape[1], B.shape[1], akm, bkm, epi, C, bias=dev(bias), res=dev(res), tile=tile)
    torch.cuda.synchronize()
    add = epi == 3
    want = x.astype(np.float64) @ y + (bias + res.astype(np.float64) if add else 0)
    mag = np.abs(x).astype(np.float64) @ np.abs(y) + (np.abs(bias) + np.abs(res) if add else 0)
    assert np.all(np.abs(C.cpu().numpy() - want) <= (K + 2) * 2.0 ** -24 * mag)


@pytest.mark.parametrize("tile", [0, 2, 3, 4])
@pytest.mark.parametrize("akm,bkm", [(0, 1), (0, 0), (1, 1)])
@pytest.mark.parametrize("small,large", [(-125, 124), (-118, 60), (-112, 0), (-100, 100)])
def test_f32_small_operands(small, large, akm, bkm, tile):
    """Operands down to the smallest normal numbers keep all their bits: 2^small times 2^large, either way round."""
    import torch
    M, N, K = 68, 132, 100
    rng = np.random.default_rng(7)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")  # noqa: E731
    for p, q in ((small, large), (large, small)):
        x, y = (np.ldexp(rng.uniform(1, 2, size=s) * rng.choice([-1, 1], size=s), e).astype(np.float32) for s, e in (((M, K), p), ((K, N), q)))
        A, B = dev(x.T if akm else x), dev(y if bkm else y.T)
        C = torch.zeros((M, N), device="cuda:0")
        print("case f32 small", p, q, akm, bkm, tile, flush=True)
        b.il_test_gemm(0, A, B, M, N, K, A.shape[1], B.shape[1], akm, bkm, 6 if akm else 0, C, tile=tile)
        torch.cuda.synchronize()
        want, mag = x.astype(np.float64) @ y, np.abs(x).astype(np.float64) @ np.abs(y)
        # 2^-149: half of it per rounding to a number below 2^-126, which the smallest pair's sums come near to
        assert np.all(np.abs(C.cpu().numpy() - want) <= (K + 2) * 2.0 ** -24 * mag + 2.0 ** -149), (p, q)
        err = np.linalg.norm(C.cpu().numpy() - want) / np.linalg.norm(want)
        assert err <= 2.0 ** -21, (p, q, err)


@pytest.mark.parametrize("tile,K", [(2, 4096), (3, 4096), (4, 4096), (0, 16384), (4, 16)])
@pytest.mark.parametrize("value", [1.0 + 2.0 ** -8 - 2.0 ** -17, 1.0038986, 1.0 - 2.0 ** -9 + 2.0 ** -18])
def test_f32_worst_split(value, tile, K):
    """Equal operands whose parts left out are the largest and of one sign: of the three products left out none is above
    2^-25 of the whole, and together they are below 2^-24.  That is the first term of the bound; the others are the
    roundings of the sum, one per product kept and addition of a K step of 16."""
    import torch
    M, N = 132, 68
    x = np.full((M, K), value, np.float32)
    y = np.full((K, N), value, np.float32)
    C = torch.zeros((M, N), device="cuda:0")
    print("case f32 worst split", value, tile, K, flush=True)
    A, B = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    b.il_test_gemm(0, A, B, M, N, K, K, N, 0, 1, 0, C, tile=tile)
    torch.cuda.synchronize()
    want = K * np.float64(np.float32(value)) ** 2
    got = C.cpu().numpy()
    assert np.all(got == got[0, 0])
    assert abs(got[0, 0] / want - 1) <= 2.0 ** -24 * (1 + 6 * -(-K // 16) + 4), got[0, 0] / want - 1


@pytest.mark.parametrize("tile,M,N,K", [(2, 130, 130, 40), (3, 130, 66, 72), (4, 68, 68, 136), (0, 67, 65, 33)])
@pytest.mark.parametrize("akm,bkm", [(0, 1), (0, 0), (1, 1)])
def test_f32_not_finite(tile, M, N, K, akm, bkm):
    """Infinities, NaN and values that round to an infinity in eight bits give what fp32 products give: an infinity
    stays one, beside rows and columns that are not touched."""
    import torch
    rng = np.random.default_rng(5)
    M, N, K = (v if tile == 0 else v // 4 * 4 for v in (M, N, K))
    x, y = (rng.normal(size=s).astype(np.float32) for s in ((M, K), (K, N)))
    y[np.abs(y) < 1e-3] = 1.0
    y[:, 0] = 1.0                                   # an operand whose rest is zero: inf * 0 must not appear
    x[0, 1], x[1, K - 1], x[2, 0], x[M - 1, 3] = np.inf, -np.inf, np.nan, 3.402e38
    y[2, N - 1], y[3, N - 1] = 0.25, 0.25           # (the large value stays finite in this column ...)
    y[3, 1] = 2.0                                   # (... and overflows in this one)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")  # noqa: E731
    A, B = dev(x.T if akm else x), dev(y if bkm else y.T)
    C = torch.zeros((M, N), device="cuda:0")
    print("case f32 not finite", tile, M, N, K, akm, bkm, flush=True)
    b.il_test_gemm(0, A, B, M, N, K, A.shape[1], B.shape[1], akm, bkm, 6 if akm else 0, C, tile=tile)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    with np.errstate(all="ignore"):
        want = x.astype(np.float64) @ y
        big = np.abs(want) > 3.4028235e38
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.isinf(got), np.isinf(want) | big) and np.all(np.sign(got[big]) == np.sign(want[big]))
        ok = np.isfinite(want) & ~big
        assert np.all(np.abs(got - want)[ok] <= ((K + 2) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(y)))[ok])


@pytest.mark.parametrize("akm,bkm,epi,beta", [(0, 1, 0, 0), (0, 1, 1, 0), (0, 1, 2, 0), (0, 0, 4, 0), (0, 0, 5, 0),
                                              (1, 1, 6, 0), (1, 1, 6, 1)])
@pytest.mark.parametrize("M,N,K", [(64, 64, 32), (37, 3, 5), (67, 132, 33), (300, 200, 260), (2816, 3000, 40)])
def test_f32_epilogues(M, N, K, akm, bkm, epi, beta):
    """Every epilogue the step has in fp32, over the tiles the library chooses and both load widths, with rows that wrap."""
    import torch
    rng = np.random.default_rng(M + 7 * N + K + epi)
    x, y = (rng.normal(size=s).astype(np.float32) for s in ((M, K), (K, N)))
    bias, c0 = rng.normal(size=N).astype(np.float32), rng.normal(size=(M, N)).astype(np.float32)
    wrap = max(1, M // 3)
    aux = rng.normal(size=(wrap, N)).astype(np.float32)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")  # noqa: E731
    A, B = dev(x.T if akm else x), dev(y if bkm else y.T)
    C, C2 = dev(c0) if beta else torch.full((M, N), float("nan"), device="cuda:0"), torch.zeros((M, N), device="cuda:0")
    print("case f32", M, N, K, akm, bkm, epi, beta, flush=True)
    b.il_test_gemm(0, A, B, M, N, K, A.shape[1], B.shape[1], akm, bkm, epi, C, C2=C2, bias=dev(bias), aux=dev(aux),
                   aux_wrap=wrap, scale=0.5, beta=beta)
    torch.cuda.synchronize()
    got = C.cpu().numpy().astype(np.float64)
    acc = x.astype(np.float64) @ y
    mag = np.abs(x).astype(np.float64) @ np.abs(y)
    bound = (K + 2) * 2.0 ** -24 * (mag + np.abs(bias) + np.abs(c0))     # K multiply-adds, two more operations
    if epi == 4:
        f = _gelu_grad(aux.astype(np.float64))[np.arange(M) % wrap]
        # the hardware's exponential and reciprocal: some 1e-6 of the derivative's terms, which reach 1.2
        assert np.all(np.abs(got - acc * f) <= bound * (1 + np.abs(f)) + 4e-6 * np.abs(acc))
        return
    want = acc + (bias if epi in (1, 2) else 0)
    if epi == 6:
        want = 0.5 * acc + (c0 if beta else 0)
    assert np.all(np.abs(got - want) <= bound)
    if epi == 2:
        g2 = C2.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(g2 - _gelu(got)) <= 4e-6 * np.abs(got) + 1e-12)


@pytest.mark.parametrize("tile", [0] + TILES)
@pytest.mark.parametrize("M,N,K,wrap", [(8, 32, 64, 8), (72, 96, 72, 40), (200, 160, 200, 200), (520, 288, 128, 130),
                                        (300, 1056, 64, 64)])
def test_row_sums_epilogue(M, N, K, wrap, tile):
    """The product of a data gradient with the sums over 32 of its columns, as stored, times another operand."""
    import torch
    rng = np.random.default_rng(M + N + K)
    x, y, aux = (_bf16(rng.standard_normal(s)) for s in ((M, K), (N, K), (wrap, N)))
    to = lambda v: torch.from_numpy(v).to(torch.bfloat16).to("cuda:0")  # noqa: E731
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    S = torch.full((M * (N // 32) + 64,), -7.0, device="cuda:0")
    print("case row sums", M, N, K, wrap, tile, flush=True)
    b.il_test_gemm(b.IL_BF16, to(x), to(y), M, N, K, K, K, 0, 0, 8, C, C2=S, aux=to(aux), aux_wrap=wrap, tile=tile)
    torch.cuda.synchronize()
    c = C.float().cpu().numpy().astype(np.float64)
    want = x.astype(np.float64) @ y.T.astype(np.float64)
    # one rounding to bf16 of a sum of K fp32 additions
    assert np.all(np.abs(c - want) <= 2.0 ** -8 * np.abs(want) + K * 2.0 ** -24 * (np.abs(x) @ np.abs(y).T))
    s = S.cpu().numpy().astype(np.float64)
    t = (c * aux[np.arange(M) % wrap]).reshape(M, N // 32, 32)
    assert np.all(np.abs(s[:M * (N // 32)].reshape(N // 32, M).T - t.sum(axis=2)) <= 32 * 2.0 ** -24 * np.abs(t).sum(axis=2))
    assert np.all(s[M * (N // 32):] == -7.0)


@pytest.mark.parametrize("streams,scale", [(1, 1.0), (2, 1.0), (2, 0.5), (2, 0.0)])
@pytest.mark.parametrize("tokens,N,K", [(64, 8, 64), (64, 264, 72), (192, 256, 128), (320, 520, 200)])
def test_gelu_gradient_with_sum_of_streams(tokens, N, K, streams, scale):
    """The FC2 data gradient of one stream, or of two whose tokens share a tile, with their weighted sum and its
    column sums; halves of the tile that end inside the operand; a stream of weight zero may hold anything."""
    import torch
    M = tokens * streams
    rng = np.random.default_rng(tokens + N + K + streams)
    x, y, aux = (_bf16(rng.standard_normal(s)) for s in ((M, K), (N, K), (tokens, N)))
    if scale == 0.0:
        x[3] = np.nan
    to = lambda v: torch.from_numpy(v).to(torch.bfloat16).to("cuda:0")  # noqa: E731
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    C2 = torch.full((tokens * N // 2 + tokens // 64 * N + 64,), -7.0, device="cuda:0")
    print("case gelu sum", tokens, N, K, streams, scale, flush=True)
    b.il_test_gemm(b.IL_BF16, to(x), to(y), M, N, K, K, K, 0, 0, 9, C, C2=C2, aux=to(aux), scale=scale, beta=streams)
    torch.cuda.synchronize()
    c = C.float().cpu().numpy().astype(np.float64).reshape(streams, tokens, N)
    f = _gelu_grad(aux.astype(np.float64))
    mag = (np.abs(x).astype(np.float64) @ np.abs(y).T.astype(np.float64)).reshape(streams, tokens, N)
    want = (x.astype(np.float64) @ y.T.astype(np.float64)).reshape(streams, tokens, N) * f
    ok = ~np.isnan(want)
    # one rounding to bf16, K fp32 additions, 1e-6 of the derivative's terms
    bound = 2.0 ** -8 * np.abs(want) + (K * 2.0 ** -24 * np.abs(f) + 4e-6) * mag
    assert np.all(np.abs(c - want)[ok] <= bound[ok]) and np.array_equal(np.isnan(c), np.isnan(want))
    w = [scale, 1.0][:streams]
    exact = sum(w[i] * c[i] if w[i] else 0 * aux.astype(np.float64) for i in range(streams))
    size = sum(abs(w[i]) * np.abs(c[i]) if w[i] else 0 * aux.astype(np.float64) for i in range(streams))
    flat = C2.cpu().numpy()
    s = C2[:tokens * N // 2].view(torch.bfloat16).float().cpu().numpy().reshape(tokens, N).astype(np.float64)
    assert np.all(np.abs(s - exact) <= 2.0 ** -8 * np.abs(exact) + 2.0 ** -23 * size)
    cols = flat[tokens * N // 2:][:tokens // 64 * N].reshape(tokens // 64, N)
    assert np.all(np.abs(cols - exact.reshape(-1, 64, N).sum(1)) <= 66 * 2.0 ** -24 * size.reshape(-1, 64, N).sum(1))
    assert np.all(flat[tokens * N // 2 + tokens // 64 * N:] == -7.0)


def _split_case(dtype, M, N, K, splits, tile, ldc):
    import torch
    rng = np.random.default_rng(M + N + K + splits)
    x, y = (_bf16(rng.standard_normal(s)) for s in ((M, K), (N, K)))
    tt = torch.float32 if dtype == b.IL_F32 else torch.bfloat16
    to = lambda v: torch.from_numpy(v).to(tt).to("cuda:0")  # noqa: E731
    C = torch.full((M, ldc), -7.0, device="cuda:0")
    ws = torch.full((splits * M * N + 64,), float("nan"), device="cuda:0")
    print("case split", dtype, M, N, K, splits, tile, flush=True)
    b.il_test_gemm_splitk(dtype, to(x), to(y), M, N, K, splits, tile, ws, C, ldc)
    torch.cuda.synchronize()
    c = C.cpu().numpy().astype(np.float64)
    want = x.astype(np.float64) @ y.T.astype(np.float64)
    bound = (K + splits) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(y).T)
    assert np.all(np.abs(c[:, :N] - want) <= bound)
    assert np.all(c[:, N:] == -7.0) and torch.isnan(ws[splits * M * N:]).all()


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K,splits", [(64, 64, 192, 2), (72, 40, 328, 3), (264, 136, 648, 5), (8, 8, 1032, 16),
                                          (64, 512, 4104, 9), (40, 24, 128, 7)])
def test_split_k_bf16(M, N, K, splits, tile):
    """Parts of whole 64-deep steps, a last part that is shorter, more parts than steps; result rows of another pitch."""
    _split_case(b.IL_BF16, M, N, K, splits, tile, N + 8)


@pytest.mark.parametrize("M,N,K,splits", [(64, 64, 192, 2), (70, 44, 333, 3), (65, 132, 260, 4), (3, 4, 1001, 16), (130, 8, 65, 2)])
def test_split_k_f32(M, N, K, splits):
    _split_case(b.IL_F32, M, N, K, splits, 0, N + 4)


@pytest.mark.parametrize("dtype", [b.IL_F32, b.IL_BF16])
@pytest.mark.parametrize("M,N,K", [(64, 64, 50304), (512, 512, 8192), (832, 768, 31992), (64, 1024, 256)])
def test_split_plan_as_the_head_takes_it(M, N, K, dtype):
    for floats in (2 ** 40, 3 * M * N, M * N, 0):
        parts, tile = b.il_gemm_split_plan(dtype, M, N, K, floats)
        assert 1 <= parts <= 32 and (parts == 1 or parts * M * N <= floats)
    parts, tile = b.il_gemm_split_plan(dtype, M, N, K, 2 ** 40)
    _split_case(dtype, M, N, K, parts, tile, N)
