"""bf16 step with both batches in one chunk (one launch for both, every layer's
weight gradient in one launch) against the same call with a chunk too small for
both together, which takes the batches one after the other: every event's
outputs bit for bit, the sums within fp32 reordering (K blocks of 16 rows summed
in fp32 in another grouping: 1e-5 of their sum of |terms|, bounded here through
the larger of the entry and the tensor's root mean square)."""
import pytest

import paper_2407_00051_amd as sg
from workloads import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,NH,d,hd8,n_theta,E,n_real", [
    (256, 1, 2, False, 1, 1, 1),              # one event each: a tile of padding, the top layer only
    (256, 3, 2, False, 2, 64, 129),           # a full tile, then a tile and one event
    (256, 4, 3, False, 1, 127, 640),          # more real than fake tiles, four layers
    (512, 2, 3, True, 3, 100, 128),
    (512, 1, 2, False, 5, 77, 5),
    (256, 2, 2, False, 30, 1000, 31000),      # enough K blocks for one launch per layer
])
def test_two_batches_match_one_by_one(gpu_ctx, H, NH, d, hd8, n_theta, E, n_real):
    print(f"case H={H} NH={NH} d={d} hd8={hd8} n_theta={n_theta} E={E} n_real={n_real}", flush=True)
    dev, n = "cuda:0", n_theta * E
    W, b = gen.xavier_mlp((8 if hd8 else d,) + (H,) * (NH + 1) + (1,), 3)
    W, b = [torch.tensor(w, device=dev) for w in W], [torch.tensor(v, device=dev) for v in b]
    th = torch.tensor(gen.theta_uniform(n_theta, d, 4), device=dev)
    real = gpu_ctx.sample_events(torch.tensor(gen.theta_uniform(1, d, 5), device=dev), n_real, 9)

    def call():
        o = gpu_ctx.disc_fwd_bwd(W, b, real, fake_source=dict(theta=th, events_per_theta=E, seed=6), precision=sg.BF16,
                                 features=sg.FEAT_HD8 if hd8 else sg.FEAT_IDENTITY)
        torch.cuda.synchronize()
        return o

    both = call()
    chunk = max((n + 127) // 128, (n_real + 127) // 128) * 128
    gpu_ctx.set_bf16_chunk_rows(chunk)
    try:
        one = call()
    finally:
        gpu_ctx.set_bf16_chunk_rows(0)
    for k in ("logits_fake", "logits_real", "dLg_dx", "dLg_dtheta"):
        assert torch.equal(both[k], one[k]), k
    pairs = [(f"dW[{l}]", both["dW"][l], one["dW"][l]) for l in range(len(W))]
    pairs += [(f"db[{l}]", both["db"][l], one["db"][l]) for l in range(len(W))]
    pairs += [(k, both[k], one[k]) for k in ("loss_d", "loss_g")]
    for k, p, q in pairs:
        scale = torch.clamp(q.abs(), min=q.square().mean().sqrt().item())
        # db_o and the first layers' sums are differences of the two batches' means
        tol = 1e-5 if k.startswith("loss") else 1e-4
        assert ((p - q).abs() <= tol * scale).all(), (k, ((p - q).abs() / scale).max().item())
