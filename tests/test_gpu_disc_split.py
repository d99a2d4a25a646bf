"""The fp32 discriminator's products on split bf16 terms: tile edges of both
tile sizes (64 events at width 128, 128 at width 64) and operands of very
different magnitudes, against the float64 oracle.

The events are a buffer, drawn away from the LeakyReLU kinks (relative margin
above 1e-6), so every output is compared tightly.  Bound of a logit: each layer
is a dot product of H terms rounded once per 8 terms (the matrix core's fp32
accumulation) and a few times more, (H / 8 + 4) 2^-24 of its sum of |terms|,
1.2e-6 at H = 128; at most four such layers, and each divides by how far its sum
cancels, which these random networks hold below 4: 2e-5.  The gradients are
products of two such chains, and their sums over events are compared against
their sums of |terms|."""
import numpy as np
import pytest

import oracle
from tests.parity import assert_condition_aware, assert_normwise, to_np
from workloads import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
LOGIT_TOL, GRAD_TOL = 2e-5, 4e-5


def _events(rng, W, b, n, d):
    """n events in (0, 1)^d with every hidden unit away from its kink."""
    kept = np.empty((0, d), dtype=np.float32)
    while len(kept) < n:
        x = rng.random((2 * n + 64, d)).astype(np.float32)
        _, pres, hs = oracle.mlp.mlp_forward(W, b, x)
        kept = np.concatenate([kept, x[oracle.mlp.kink_margin(W, b, hs, pres[:-1]) > 1e-6]])
    return kept[:n]


@pytest.mark.parametrize("H,NH,d,n_fake,n_real,scale", [
    (64, 1, 2, 1, 1, 1.0), (64, 1, 2, 127, 129, 1.0), (64, 2, 3, 128, 65, 1.0), (64, 3, 2, 193, 64, 1.0),
    (128, 1, 2, 63, 65, 1.0), (128, 2, 2, 64, 1, 1.0), (128, 2, 3, 65, 127, 1.0), (128, 2, 2, 64 * 260 + 1, 64 * 3, 1.0),
    # one hidden layer's operands small and the next one's large: the terms keep
    # their relative size, so the result only scales
    (128, 2, 2, 130, 70, 1e-12), (64, 3, 2, 130, 70, 1e12),
])
def test_split_products(gpu_ctx, H, NH, d, n_fake, n_real, scale):
    print(f"case H={H} NH={NH} d={d} n_fake={n_fake} n_real={n_real} scale={scale}", flush=True)
    rng = np.random.default_rng(17)
    W, b = gen.xavier_mlp((d,) + (H,) * (NH + 1) + (1,), 5)
    s = np.float32(scale)
    W[1], b[1] = W[1] * s, b[1] * s
    if NH > 1:
        W[2] = W[2] / s
    fake, real = _events(rng, W, b, n_fake, d), _events(rng, W, b, n_real, d)
    dev = "cuda:0"
    o = gpu_ctx.disc_fwd_bwd([torch.tensor(w, device=dev) for w in W], [torch.tensor(v, device=dev) for v in b],
                             torch.tensor(real, device=dev), fake_x=torch.tensor(fake, device=dev))
    torch.cuda.synchronize()
    ref = oracle.disc_fwd_bwd(W, b, fake.astype(np.float64), real.astype(np.float64))
    assert_normwise(to_np(o["logits_fake"]), ref["logits_fake"], LOGIT_TOL, "logits_fake")
    assert_normwise(to_np(o["logits_real"]), ref["logits_real"], LOGIT_TOL, "logits_real")
    for l in range(len(W)):
        assert_condition_aware(to_np(o["dW"][l]), ref["dW"][l], ref["dW_cond"][l], GRAD_TOL, f"dW[{l}]")
        assert_condition_aware(to_np(o["db"][l]), ref["db"][l], ref["db_cond"][l], GRAD_TOL, f"db[{l}]")
    assert_normwise(to_np(o["dLg_dx"]), ref["dLg_din"], GRAD_TOL, "dLg_dx")
