"""bf16 step with both batches in one chunk (one launch for both) against the same
call with a chunk too small for both together, which takes the batches one after
the other, in one chunk each or in several: every event's outputs bit for bit, the
sums within fp32 reordering (K blocks of 16 rows summed in fp32 in another grouping:
1e-5 of their sum of |terms|, bounded here through the larger of the entry and the
tensor's root mean square).

A chunk's weight gradients take every layer in one launch where the chunk has fewer
K blocks (of 16 rows) than 32 times the CUs per layer and 256 x 256 tile, else a
launch per layer, whose partials share one buffer.  Each case says which of the two
either side takes, and that is checked against the sizes."""
import pytest

import paper_2407_00051_amd as sg
from workloads import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _one_launch(H, NH, rows):
    """Whether a chunk of so many (padded) rows takes all layers in one launch."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return rows // 16 < 32 * max(1, cus // ((H // 256) ** 2 * NH))


@pytest.mark.parametrize("H,NH,d,hd8,n_theta,E,n_real,chunk,both_one,single_one", [
    (256, 1, 2, False, 1, 1, 1, 0, True, True),            # one event each: a tile of padding, the top layer only
    (256, 3, 2, False, 2, 64, 129, 0, True, True),         # a full tile, then a tile and one event
    (256, 4, 3, False, 1, 127, 640, 0, True, True),        # more real than fake tiles, four layers
    (512, 2, 3, True, 3, 100, 128, 0, True, True),
    (512, 1, 2, False, 5, 77, 5, 0, True, True),
    (256, 2, 2, False, 30, 1000, 31000, 0, True, True),    # 3,824 and 1,944 K blocks of 4,096
    (256, 2, 2, False, 40, 1000, 40001, 0, False, True),   # 5,008 and 2,504 of 4,096
    (512, 3, 3, True, 3, 2033, 6111, 0, False, True),      # 768 and 384 of 672
    (512, 3, 2, False, 12, 1000, 12345, 0, False, False),  # 1,528 and 776 of 672
    (256, 3, 2, False, 30, 3001, 77777, 46080, False, False),   # 10,496 of 2,720; chunks of 2,880, two a batch
    (512, 3, 3, False, 30, 1000, 25000, 12800, False, False),   # 3,448 of 672; chunks of 800, three and two
])
def test_two_batches_match_one_by_one(gpu_ctx, H, NH, d, hd8, n_theta, E, n_real, chunk, both_one, single_one):
    print(f"case H={H} NH={NH} d={d} hd8={hd8} n_theta={n_theta} E={E} n_real={n_real} chunk={chunk}", flush=True)
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

    pad = [(k + 127) // 128 * 128 for k in (n, n_real)]
    chunk = chunk or max(pad)
    assert (_one_launch(H, NH, sum(pad)), _one_launch(H, NH, chunk)) == (both_one, single_one) and sum(pad) > chunk
    both = call()
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
