"""The generator's 64-row forward kernel (split bf16 products, taken when 64-row
tiles of all members cover the CUs) at the edges of its tiles, depths and input
and output widths, against the float64 oracle.

theta = 1 + softplus(o) >= 1, so an elementwise relative bound: each hidden layer
rounds its sum once per 8 products and a few times more, (128 / 8 + 4) 2^-24 of its
sum of |terms| (1.2e-6), at most four layers feed one another, and softplus' <= 1:
2e-5 covers them with a factor for sums that cancel."""
import numpy as np
import pytest

import oracle
from tests.parity import to_np
from workloads import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("widths,M,k", [
    ((6, 128, 128, 128, 128, 6), 256, 1),       # one row of a tile
    ((6, 128, 128, 128, 128, 6), 130, 65),      # a full tile and one row; members past the last multiple of 8
    ((7, 128, 128, 128, 1), 128, 127),          # in > 6, one output
    ((1, 128, 128, 8), 3, 64 * 86),             # one hidden-to-hidden layer, whole tiles
    ((8, 128, 128, 128, 128, 8), 86, 192),
])
def test_gen_forward_split(gpu_ctx, widths, M, k):
    print(f"case gen forward widths={widths} M={M} k={k}", flush=True)
    W, b = gen.generator_stack(widths, M, seed=len(widths) + k)
    n = gen.noise(k, widths[0], seed=k + 3)
    dev = "cuda:0"
    th = gpu_ctx.gen_forward([torch.tensor(w, device=dev) for w in W], [torch.tensor(v, device=dev) for v in b],
                             torch.tensor(n, device=dev))
    torch.cuda.synchronize()
    got, worst = to_np(th).astype(np.float64), 0.0
    for m in sorted({m for m in (0, 1, 7, M // 2, M - 2, M - 1) if m < M}):
        ref = oracle.generator_forward([w[m] for w in W], [v[m] for v in b], n)
        worst = max(worst, float(np.max(np.abs(got[m] - ref) / np.abs(ref))))
    print(f"  worst relative error {worst:.2e}", flush=True)
    assert worst <= 2e-5


@pytest.mark.parametrize("M,k", [(129, 5), (300, 37)])   # more members than a slice keeps; rows past the last block
def test_ensemble_statistics_of_many_members(gpu_ctx, M, k):
    print(f"case ensemble M={M} k={k}", flush=True)
    W, b = gen.generator_stack((6, 128, 128, 6), M, seed=M)
    n = gen.noise(k, 6, seed=k)
    dev = "cuda:0"
    o = gpu_ctx.ensemble_response([torch.tensor(w, device=dev) for w in W], [torch.tensor(v, device=dev) for v in b],
                                  torch.tensor(n, device=dev))
    torch.cuda.synchronize()
    p_hat, sigma = oracle.ensemble_response(
        np.stack([oracle.generator_forward([w[m] for w in W], [v[m] for v in b], n) for m in range(M)]))
    # each theta within 2e-5 (above), and the means of M k of them no further
    np.testing.assert_allclose(to_np(o["p_hat"]), p_hat, rtol=2e-5)
    np.testing.assert_allclose(to_np(o["sigma"]), sigma, rtol=2e-5, atol=2e-5 * np.abs(p_hat).max())


def test_gen_forward_split_nonfinite_rows(gpu_ctx):
    """An infinite or NaN noise value makes its row's output NaN for every member and leaves
    the other rows bit for bit."""
    print("case gen forward non-finite", flush=True)
    M, k, dev = 130, 150, "cuda:0"
    W, b = gen.generator_stack((6, 128, 128, 128, 128, 6), M, seed=9)
    W, b = [torch.tensor(w, device=dev) for w in W], [torch.tensor(v, device=dev) for v in b]
    n = torch.tensor(gen.noise(k, 6, seed=4), device=dev)
    clean = gpu_ctx.gen_forward(W, b, n)
    v = n.clone()
    v[3, 2], v[64, 0], v[149, 5] = float("inf"), float("nan"), float("-inf")
    th = gpu_ctx.gen_forward(W, b, v)
    torch.cuda.synchronize()
    good = torch.ones(k, dtype=torch.bool, device=dev)
    good[torch.tensor([3, 64, 149], device=dev)] = False
    assert torch.isnan(th[:, ~good]).all()
    assert torch.equal(th[:, good], clean[:, good])
