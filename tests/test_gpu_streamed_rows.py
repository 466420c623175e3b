"""GPU parity of the streamed expert kernels (few token rows per expert): the lane layouts of a row (whole and padded, in
one wave and shared by four), items of one to eight rows and experts that take several, both pagers, fp8 and
bf16, against the oracle, and bit for bit against the resident run and (to four tokens) the device pager; and, by the
launches counted, that these kernels run on one side of their lines and not on the other."""
import ctypes

import numpy as np
import pytest

import oracle
from parity import log, run_case
from paper_2606_21868_amd import wisp
from paper_2606_21868_amd.workloads import FP8, ROUTE_SIGMOID_GROUP, WORKLOADS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BF16 = WORKLOADS["qwen3-30b-a3b-decode"]
F8 = BF16.with_(w_dtype=FP8, route=ROUTE_SIGMOID_GROUP, n_groups=4, topk_groups=2, has_shared=True)

# (workload, cap, steps, streamed): lanes x chunks per lane (x waves) of gate/up and of down, "+" where padded.  Every layout
# runs in bf16 in at least one of the two products (one chunk
# per lane only in down: layers whose gate/up rows are so short stay per item).
CASES = {
    # up to four tokens: the device pager runs the same rows (checked bit for bit by run_case)
    "fp8 64x7 16x1, one token, both pagers": (F8.with_(L=2, T=1, d=7168, I=256, N=16, k=4), 5, 6, True),
    "fp8 64x7 64x2, four tokens, both pagers": (F8.with_(L=1, T=4, d=7168, I=2048, N=16, k=4), 16, 2, True),
    "bf16 64x4 32x3, three tokens, both pagers": (BF16.with_(L=2, T=3, d=2048, I=768, N=32, k=4), 12, 4, True),
    # an expert of 15 rows (two items), a shared expert
    "bf16 64x3+ 32x3+, shared": (BF16.with_(L=2, T=15, d=1472, I=704, N=12, k=3, has_shared=True), 5, 2, True),
    "bf16 64x2 64x3": (BF16.with_(L=1, T=9, d=1024, I=1536, N=8, k=2), 4, 1, True),
    "bf16 64x5 32x5": (BF16.with_(L=1, T=6, d=2560, I=1280, N=8, k=2), 4, 1, True),
    "bf16 64x7 64x6": (BF16.with_(L=1, T=4, d=3584, I=3072, N=6, k=2), 4, 1, True),
    "bf16 64x8 64x2+": (BF16.with_(L=1, T=3, d=4096, I=960, N=6, k=2), 4, 1, True),
    "bf16 32x3 64x4": (BF16.with_(L=1, T=8, d=768, I=2048, N=8, k=3), 4, 1, True),
    "bf16 32x5+ 32x5+": (BF16.with_(L=1, T=7, d=1088, I=1088, N=8, k=2), 4, 1, True),
    "bf16 16x3 64x6": (BF16.with_(L=1, T=8, d=384, I=3072, N=8, k=2), 4, 1, True),
    # rows shared by four waves, whole and padded (a last wave with little or nothing of the row)
    "bf16 64x3x4+ 64x4x4": (BF16.with_(L=1, T=5, d=5120, I=8192, N=4, k=2), 4, 1, True),
    "bf16 64x3x4 16x3": (BF16.with_(L=1, T=9, d=6144, I=384, N=6, k=2), 4, 1, True),
    "bf16 64x4x4 16x1": (BF16.with_(L=1, T=2, d=8192, I=128, N=6, k=2), 4, 1, True),
    "bf16 64x5x4 32x5+": (BF16.with_(L=1, T=4, d=10240, I=1088, N=4, k=2), 4, 1, True),
    "bf16 64x6x4+ 64x1": (BF16.with_(L=1, T=3, d=11264, I=512, N=4, k=2), 4, 1, True),
    "bf16 64x8x4 32x1": (BF16.with_(L=1, T=6, d=16384, I=256, N=4, k=2), 4, 1, True),
    "bf16 64x8 64x7x4": (BF16.with_(L=1, T=5, d=4096, I=14336, N=3, k=2), 3, 1, True),
    # fp8
    "fp8 64x3+ 16x3": (F8.with_(L=1, T=7, d=2944 - 256, I=768, N=16, k=4), 8, 2, True),
    "fp8 64x2 32x3+": (F8.with_(L=1, T=5, d=2048, I=1408, N=16, k=4), 8, 1, True),
    "fp8 64x5 32x3": (F8.with_(L=1, T=2, d=5120, I=1536, N=8, k=2), 4, 1, True),
    "fp8 64x3x4+ 16x1": (F8.with_(L=1, T=3, d=10240, I=256, N=8, k=2), 4, 1, True),
    "fp8 64x4x4 64x1": (F8.with_(L=1, T=9, d=16384, I=1024, N=4, k=2), 4, 1, True),
    # the other side of the line: small layers stay on the per-item kernels (with either pager), and widths whose padding
    # would be a quarter or more
    "fp8 four tokens, both pagers": (F8.with_(L=1, T=4, d=256, I=2048, N=16, k=4), 16, 3, False),
    "bf16 three tokens, both pagers": (BF16.with_(L=2, T=3, d=384, I=768, N=32, k=4), 12, 4, False),
    "bf16 two tokens, both pagers": (BF16.with_(L=1, T=2, d=2048, I=128, N=16, k=8), 16, 3, False),
    "bf16 short rows": (BF16.with_(L=1, T=9, d=128, I=320, N=24, k=6), 7, 2, False),
    "bf16 refused width": (BF16.with_(L=1, T=5, d=4608, I=1024, N=4, k=2), 4, 1, False),
    "fp8 refused width": (F8.with_(L=1, T=5, d=7168, I=384, N=8, k=2), 4, 1, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_streamed_rows(name):
    wl, cap, steps, streamed = CASES[name]
    run_case(wl, cap, steps, check_all_outputs=True, expect_grouped=False, expect_streamed=streamed)


# token batches on both sides of the line: evenly routed with few and with more rows per expert, with a shared expert (its
# tokens stream too) and, from 128 experts and more, more items than a launch takes and experts of more than eight rows;
# layers of short rows never stream
@pytest.mark.parametrize("T,N,k,d,I,shared,streamed", [
    (20, 64, 4, 768, 256, False, True), (100, 64, 4, 768, 256, False, False), (16, 60, 6, 1472, 704, True, True),
    (30, 60, 6, 1472, 704, True, True), (50, 60, 6, 1472, 704, True, False), (120, 230, 8, 768, 128, False, True),
    (17, 24, 2, 5120, 128, False, True), (16, 8, 2, 256, 128, False, False), (40, 16, 2, 256, 256, False, False),
    (41, 16, 2, 256, 256, False, False), (33, 12, 1, 320, 192, True, False), (120, 230, 8, 256, 128, False, False)])
def test_streamed_token_batches(T, N, k, d, I, shared, streamed):
    wl = WORKLOADS["qwen3-30b-a3b-prefill"].with_(L=1, T=T, N=N, k=k, d=d, I=I, has_shared=shared)
    run_case(wl, max(1, N // 3), 1, check_all_outputs=True, expect_grouped=True, expect_streamed=streamed)


def test_token_batch_with_skewed_routing_runs_grouped():
    # every token on the same four of 64 experts: few rows per expert of the layer, many per expert that is used
    wl = WORKLOADS["qwen3-30b-a3b-prefill"].with_(L=1, T=40, N=64, k=4, d=768, I=256)
    log("[case] skewed routing")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        run.set_cap(16)
        ids = np.tile(np.array([3, 17, 40, 41], np.int32), (wl.T, 1))
        g = torch.full((wl.T, wl.k), 0.25, device=run.dev)
        y = torch.zeros((wl.T, wl.d), device=run.dev)
        run.ctx.set_profiling(1 << wisp.K_GROUPED_GATEUP)
        run.ctx.page_in(0, ids, wl.T)
        run.ctx.moe_forward(0, run.x_dev[0, 0], wl.T, g, y, run.stream)
        run.stream.synchronize()
        run.ctx.set_profiling(0)
        assert run.ctx.kernel_times(wisp.K_GROUPED_GATEUP)["launches"] > 0 == run.ctx.kernel_times(wisp.K_STREAMED)["launches"]
        want = np.stack([sum(0.25 * oracle.expert(run.master_ptrs(0)[e], wl.w_dtype, wl.d, wl.I, run.x_host[0, 0, t]) for e in ids[0])
                         for t in range(wl.T)])
        err = np.abs(y.cpu().numpy() - want).max(-1) / np.abs(want).max(-1)
        assert err.max() <= 2e-2, err.max()
    finally:
        run.close()


@pytest.mark.parametrize("name", ["bf16 64x3+ 32x3+, shared", "fp8 64x3+ 16x3"])
def test_offload_arm_streams_the_same_bits(name):
    # the static-offload arm builds its items from work lists; an expert of more than eight rows among them
    wl = CASES[name][0].with_(L=1)
    log(f"[case] offload arm {name}")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        run.set_cap(wl.N)
        run.ctx.preload()
        ref = run.decode(record=True, steps=1)
        run.ctx.offload_begin(wl.N * ((run.blob_bytes + 4095) // 4096 * 4096), wisp.OFFLOAD_ZERO_COPY)
        run.ctx.set_profiling(1 << wisp.K_FFN_GATEUP)
        out = run.offload(record=True, steps=1)
        run.ctx.set_profiling(0)
        run.ctx.offload_end()
        assert run.ctx.kernel_times(wisp.K_STREAMED)["launches"] > 0
        assert np.array_equal(out["idx"], ref["idx"])
        assert np.array_equal(out["y"].view(np.uint32), ref["y"].view(np.uint32))
    finally:
        run.close()


# Rows whose chunks do not fill their lanes (in one wave, over four waves, fp8), with an infinite weight or block scale in the
# last chunk: what lies past a row's end must not turn the infinity into a NaN.  One expert alone holds infinities; fp8 codes and
# inputs are made positive so that every infinite term has one sign.
@pytest.mark.parametrize("wl", [BF16.with_(L=1, T=3, d=1472, I=704, N=6, k=2), BF16.with_(L=1, T=2, d=5120, I=1472, N=4, k=2),
                                F8.with_(L=1, T=2, d=2688, I=1920, N=4, k=2, n_groups=2, topk_groups=2, has_shared=False)],
                         ids=["bf16 one wave", "bf16 four waves", "fp8"])
@pytest.mark.parametrize("matrix", ["W3", "W2"])
def test_infinities_in_padded_rows(wl, matrix):
    log(f"[case] infinity in {matrix} d={wl.d} I={wl.I} w={wl.w_dtype}")
    d, I, n = wl.d, wl.I, wl.d * wl.I
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        if wl.w_dtype == FP8:
            run.x_host &= 0x7FFF
            run.x_dev &= 0x7FFF
        first = oracle.route(wl.route, run.wr_host[0], run.x_host[0, 0, 0], wl.k, wl.n_groups, wl.topk_groups)[0][0]
        for e in range(wl.N):
            ptr, nbytes = run.ctx.expert_host_ptr(0, e)
            raw = np.ctypeslib.as_array((ctypes.c_uint8 * nbytes).from_address(ptr))
            if wl.w_dtype == FP8:
                raw[:3 * n] &= 0x7F   # positive codes
                s1, s3, s2 = np.split(raw[3 * n:].view(np.uint16), 3)
                if e == first:
                    (s3 if matrix == "W3" else s2)[(d if matrix == "W3" else I) // 128 - 1] = 0x7F80   # the first rows' last block
                    raw[:3 * n][raw[:3 * n] == 0] = 0x08   # no zero codes: 0 times an infinite scale is no number
            elif e == first:
                w = raw.view(np.uint16)
                w[n + d - 1 if matrix == "W3" else 2 * n + I - 1] = 0x7F80   # the last weight of row 0
        run.ctx.masters_ready()
        assert run.set_cap(wl.N) == wl.N
        out = run.decode(record=True, steps=1)
        idx, _, y, _, _ = oracle.moe_layer(wl.route, run.master_ptrs(0), run.wr_host[0], run.x_host[0, 0], wl.k, wl.I,
                                           wl.w_dtype, None, wl.n_groups, wl.topk_groups)
        got = out["y"][0, 0].astype(np.float64)
        assert np.array_equal(idx, out["idx"][0, 0])
        assert np.isinf(y).any() and not np.isnan(y).any()
        assert np.array_equal(np.isnan(got), np.isnan(y)) and np.array_equal(np.isinf(got), np.isinf(y))
        assert np.array_equal(np.sign(got[np.isinf(y)]), np.sign(y[np.isinf(y)]))
        fin = np.where(np.isinf(y), 0.0, y)
        err = np.abs(np.where(np.isinf(y), 0.0, got) - fin).max(-1) / np.maximum(np.abs(fin).max(-1), 1e-30)
        assert err.max() <= 2e-2, err
    finally:
        run.close()
