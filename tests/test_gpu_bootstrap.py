"""GPU parity of the bootstrap draw (sagips_bootstrap) against the oracle,
through the C ABI: drawn rows bit-exact, gathered values exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_00051_amd as sg  # noqa: E402


@pytest.mark.parametrize("n_data,d,n_out,seed,step", [
    (1, 2, 100, 0, 0),                  # a single row
    (1000, 2, 777, 5, 3),               # ragged sizes
    (4096, 3, 10000, 7, 123456),        # d = 3, a power-of-two row count, more draws than rows
    (3_000_017, 2, 1_500_008, 2**40 + 11, 2**32 - 1),   # 64-bit seed, the largest step
])
def test_bootstrap_matches_oracle(gpu_ctx, n_data, d, n_out, seed, step):
    print(f"case bootstrap n_data={n_data} d={d} n_out={n_out}", flush=True)
    rng = np.random.default_rng(n_data)
    data_np = rng.standard_normal((n_data, d)).astype(np.float32)
    data = torch.tensor(data_np, device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, seed, step, want_idx=True)
    torch.cuda.synchronize()
    ref_idx = oracle.bootstrap_indices(n_data, n_out, seed, step)
    got = idx.cpu().numpy()
    assert np.array_equal(got, ref_idx), np.flatnonzero(got != ref_idx)[:10]
    assert np.array_equal(out.cpu().numpy(), data_np[ref_idx])


def test_bootstrap_full_size_sampled(gpu_ctx):
    """Medium-size reference data (8,388,608 events) and a 50% draw: every drawn
    row checked, at the launch configuration the benchmark times."""
    n_data, n_out = 1 << 23, 1 << 22
    data = torch.randn((n_data, 2), device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, 2024, 17, want_idx=True)
    torch.cuda.synchronize()
    ref_idx = oracle.bootstrap_indices(n_data, n_out, 2024, 17)
    assert np.array_equal(idx.cpu().numpy(), ref_idx)
    assert torch.equal(out, data[torch.tensor(ref_idx, device="cuda:0")])
    # the variant without the index output (the one the benchmark times) draws the same rows
    assert torch.equal(gpu_ctx.bootstrap(data, n_out, 2024, 17), out)


def test_bootstrap_three_observable_full_size(gpu_ctx):
    """Three-observable reference data at full size (33,554,432 events, 16,777,216 draws)."""
    n_data, n_out = 1 << 25, 1 << 24
    data = torch.randn((n_data, 3), device="cuda:0")
    out = gpu_ctx.bootstrap(data, n_out, 99, 4)
    torch.cuda.synchronize()
    ref_idx = torch.tensor(oracle.bootstrap_indices(n_data, n_out, 99, 4), device="cuda:0")
    assert torch.equal(out, data[ref_idx])


def test_bootstrap_rejects_bad_arguments(gpu_ctx):
    data = torch.zeros((100, 2), device="cuda:0")
    with pytest.raises(sg.SagipsError):
        gpu_ctx.bootstrap(data, 0, 1, 1)
    with pytest.raises(ValueError):
        gpu_ctx.bootstrap(torch.zeros((100, 4), device="cuda:0"), 10, 1, 1)
    # out overlapping data is refused before any launch
    with pytest.raises(sg.SagipsError):
        gpu_ctx.bootstrap(data, 50, 1, 1, out=data[:50])


@pytest.mark.parametrize("n_data,d,n_out,seed,step", [
    (1, 2, 100, 0, 0),                  # one slab, one row drawn 100 times
    (1000, 2, 777, 5, 3),               # ragged
    (4096, 3, 10000, 7, 123456),        # more draws than rows
    (16384 * 3 + 5, 2, 70001, 11, 9),   # a partial last slab
    (3_000_017, 2, 1_500_008, 2**40 + 11, 2**32 - 1),
])
def test_bootstrap_row_order_matches_oracle(gpu_ctx, n_data, d, n_out, seed, step):
    print(f"case bootstrap rows n_data={n_data} d={d} n_out={n_out}", flush=True)
    rng = np.random.default_rng(n_data + 1)
    data_np = rng.standard_normal((n_data, d)).astype(np.float32)
    data = torch.tensor(data_np, device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, seed, step, want_idx=True, row_order=True)
    torch.cuda.synchronize()
    ref_x, ref_idx = oracle.bootstrap_row_order(data_np, n_out, seed, step)
    assert np.array_equal(idx.cpu().numpy(), ref_idx)
    assert np.array_equal(out.cpu().numpy(), ref_x)


@pytest.mark.parametrize("n_data,d,n_out", [(1 << 23, 2, 1 << 22), (1 << 25, 3, 1 << 24)])
def test_bootstrap_row_order_full_size(gpu_ctx, n_data, d, n_out):
    """The benchmarked sizes: the row-order sample is the draw-order sample's
    multiset (per-row counts), in ascending order, with the rows' values."""
    data = torch.randn((n_data, d), device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, 31, 6, want_idx=True, row_order=True)
    _, draws = gpu_ctx.bootstrap(data, n_out, 31, 6, want_idx=True)
    assert torch.equal(torch.bincount(idx, minlength=n_data), torch.bincount(draws, minlength=n_data))
    assert bool((idx[1:] >= idx[:-1]).all())
    assert torch.equal(out, data[idx])
    # without the index output
    assert torch.equal(gpu_ctx.bootstrap(data, n_out, 31, 6, row_order=True), out)


@pytest.mark.parametrize("n_data,n_out", [
    # the draws are sorted in 1,024 chunks at most, 40,960 draws at a time: more than
    # 41,943,040 draws take two batches a chunk, the second one short ...
    (100_003, 1024 * 40960 + 12_345),
    # ... or two nearly full ones and a ragged last chunk
    (5_000_011, 2 * 1024 * 40960 - 77),
    ((1 << 27) - 5, 3_000_001),          # 8,192 slabs of 16,384 rows, the most there can be, the last one partial
    ((1 << 25) + 1, 1_000_003),          # 2,049 slabs: one more than two per thread
])
def test_bootstrap_row_order_beyond_one_batch(gpu_ctx, n_data, n_out):
    """As test_bootstrap_row_order_full_size, at the largest tables and draw counts."""
    print(f"case bootstrap rows n_data={n_data} n_out={n_out}", flush=True)
    data = torch.randn((n_data, 2), device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, 2**35 + 3, 8, want_idx=True, row_order=True)
    _, draws = gpu_ctx.bootstrap(data, n_out, 2**35 + 3, 8, want_idx=True)
    assert torch.equal(torch.bincount(idx, minlength=n_data), torch.bincount(draws, minlength=n_data))
    assert bool((idx[1:] >= idx[:-1]).all())
    assert torch.equal(out, data[idx])


@pytest.mark.parametrize("n_data,d,n_out,sort", [
    (64 << 14, 2, 1020, False),          # one chunk, either side of the least run it is sorted from
    (64 << 14, 3, 1021, True),
    ((2048 << 14) + 1, 2, 1001, False),  # 2,049 slabs, most of them without a draw
    ((2048 << 14) + 1, 2, 4_194_305, True),
    ((1 << 27) - 5, 2, 5_000_001, False),
    ((1 << 27) - 5, 2, 1 << 24, True),   # 8,192 slabs sorted: exactly four draws of a slab and chunk
    ((1 << 27) - 5, 2, (1 << 24) + 1, False),
])
def test_bootstrap_row_order_both_scatters(gpu_ctx, n_data, d, n_out, sort):
    """As test_bootstrap_row_order_full_size, on both sides of the rule that sorts a chunk's
    draws by slab before they are written."""
    print(f"case bootstrap rows n_data={n_data} n_out={n_out}", flush=True)
    slabs = -(-n_data // 16384)
    chunks = max(1, min(1024, max(-(-n_out // 32768), min(256, -(-n_out // 16384)))))
    least = 16.0 - 12.5 * chunks / 256 if chunks <= 256 else 4.0
    assert (min(-(-n_out // chunks), 40960) >= least * slabs) == sort
    data = torch.randn((n_data, d), device="cuda:0")
    out, idx = gpu_ctx.bootstrap(data, n_out, 77, 2, want_idx=True, row_order=True)
    _, draws = gpu_ctx.bootstrap(data, n_out, 77, 2, want_idx=True)
    assert torch.equal(idx, draws.sort().values)
    assert torch.equal(out, data[idx])


def test_bootstrap_row_order_limits(gpu_ctx):
    data = torch.zeros((100, 2), device="cuda:0")
    big = torch.zeros(((1 << 27) + 1, 2), device="cuda:0")
    with pytest.raises(sg.SagipsError):
        gpu_ctx.bootstrap(big, 10, 1, 1, row_order=True)
    del big
    with pytest.raises(sg.SagipsError):
        gpu_ctx.bootstrap(data, 0, 1, 1, row_order=True)
