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
