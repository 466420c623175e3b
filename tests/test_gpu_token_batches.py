"""GPU parity of token batches with fp8 weights, other widths than the bf16 grouped GEMMs take, or a shared
expert: against the oracle, and bit for bit against the resident run and the static-offload arms."""
import numpy as np
import pytest

from parity import log, run_case
from paper_2606_21868_amd import wisp
from paper_2606_21868_amd.workloads import FP8, ROUTE_SIGMOID_GROUP, WORKLOADS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BF16_BATCH = WORKLOADS["qwen3-30b-a3b-prefill"]
FP8_BATCH = BF16_BATCH.with_(w_dtype=FP8, route=ROUTE_SIGMOID_GROUP, n_groups=4, topk_groups=2, has_shared=True)

# (workload, cap): row blocks with a remainder, experts of one row and of two row blocks, tiles shorter than
# the loads run ahead (K of one to three stages), columns that end inside a tile
CASES = {
    # fp8: ~20 rows per expert and a shared expert of 83 (two row blocks of 64); down of two stages
    "fp8": (FP8_BATCH.with_(L=2, T=83, d=384, I=256, N=16, k=4), 5),
    # fp8, single-stage K in the down product, ~130 rows: the wide tiles, two row blocks of 128
    "fp8 wide": (FP8_BATCH.with_(L=1, T=260, d=512, I=128, N=8, k=4), 3),
    # the smallest batch on this path: experts of one or two rows
    "fp8 few rows": (FP8_BATCH.with_(L=2, T=16, d=256, I=256, N=64, k=4), 20),
    # bf16, widths that are multiples of 64 only (a last tile of one wave), with a shared expert
    "bf16 shared": (BF16_BATCH.with_(L=2, T=37, d=320, I=192, N=12, k=3, has_shared=True), 5),
    # more tiles than workgroups, by a part of a round (704 and 768 tiles over 512 when all experts are resident)
    "bf16 partial round": (BF16_BATCH.with_(L=1, T=203, d=1472, I=704, N=60, k=6, has_shared=True), 20),
    # bf16, the same widths without one, K of one stage, wide tiles with a last column tile of half a tile
    "bf16 wide": (BF16_BATCH.with_(L=1, T=500, d=320, I=64, N=8, k=2), 3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_token_batch_parity(name):
    wl, cap = CASES[name]
    out = run_case(wl, cap, 1, check_all_outputs=True, expect_grouped=True)
    assert out["chunks"].min() >= 2


def test_token_batch_more_experts_than_a_launch_takes():
    # 200 experts of ~3 rows plus the shared one: two launches
    wl = BF16_BATCH.with_(L=1, T=150, d=128, I=64, N=200, k=4, has_shared=True)
    run_case(wl, 200, 1, check_all_outputs=True, expect_grouped=True)


@pytest.mark.parametrize("name", ["fp8", "bf16 shared"])
def test_token_batch_offload_arms_give_the_same_bits(name):
    wl, _ = CASES[name]
    log(f"[case] offload arms {name} T={wl.T}")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        run.set_cap(wl.N)
        run.ctx.preload()
        ref = run.decode(record=True, steps=1)
        layer = wl.N * ((run.blob_bytes + 4095) // 4096 * 4096)
        for mode, budget in ((wisp.OFFLOAD_ZERO_COPY, layer), (wisp.OFFLOAD_BULK, 2 * layer)):
            run.ctx.offload_begin(budget, mode)
            try:
                out = run.offload(record=True, steps=1)
            finally:
                run.ctx.offload_end()
            assert np.array_equal(out["idx"], ref["idx"]), mode
            assert np.array_equal(out["y"].view(np.uint32), ref["y"].view(np.uint32)), mode
    finally:
        run.close()


@pytest.mark.parametrize("name", ["fp8", "bf16 shared"])
def test_token_batch_at_any_address(name):
    # hidden states two bytes past a 16-byte boundary: the direct-to-LDS loads do not take them, the per-item kernels do
    wl, cap = CASES[name]
    log(f"[case] unaligned rows {name} T={wl.T}")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        run.set_cap(cap)
        ref = run.decode(record=True, steps=1)
        n = run.x_dev.numel()
        off = torch.zeros(n + 8, dtype=run.x_dev.dtype, device=run.dev)[1:1 + n].view(run.x_dev.shape)
        assert off.data_ptr() % 16 == 2 and off.is_contiguous()
        off.copy_(run.x_dev)
        run.x_dev = off
        run.ctx.set_profiling(1 << wisp.K_GROUPED_GATEUP)
        out = run.decode(record=True, steps=1)
        run.ctx.set_profiling(0)
        assert run.ctx.kernel_times(wisp.K_GROUPED_GATEUP)["launches"] == 0
        assert np.array_equal(out["idx"], ref["idx"]) and np.array_equal(out["w"], ref["w"])
        err = np.abs(out["y"] - ref["y"]).max(-1) / np.abs(ref["y"]).max(-1)
        assert err.max() <= 4e-2, err.max()   # each within 2e-2 of the oracle's row (parity.tolerance)
    finally:
        run.close()


@pytest.mark.parametrize("name", ["fp8", "bf16 shared"])
def test_forward_with_given_ids_does_not_wait_for_the_stream(name):
    # page-in and forward with ids of the caller's own (no routing call): the host runs ahead of the stream, as with few tokens
    wl, _ = CASES[name]
    log(f"[case] forwards ahead of the stream {name} T={wl.T}")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        run.set_cap(wl.N)
        run.ctx.preload()
        ids = [np.stack([(np.arange(wl.k) + t + 3 * l) % wl.N for t in range(wl.T)]).astype(np.int32) for l in range(wl.L)]
        g = torch.full((wl.T, wl.k), 1.0 / wl.k, device=run.dev)
        y = torch.zeros((3, wl.L, wl.T, wl.d), device=run.dev)
        a = torch.zeros((8192, 8192), dtype=torch.bfloat16, device=run.dev)
        busy = torch.cuda.Event()

        def step(i):
            for l in range(wl.L):
                run.ctx.page_in(l, ids[l], wl.T)
                run.ctx.moe_forward(l, run.x_dev[0, l], wl.T, g, y[i, l], run.stream)
        step(0)
        torch.cuda.synchronize()
        with torch.cuda.stream(run.stream):
            for _ in range(60):   # tens of milliseconds
                a @ a
            busy.record()
        step(1)
        assert not busy.query()
        step(2)
        torch.cuda.synchronize()
        assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])
    finally:
        run.close()
