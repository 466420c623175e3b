"""GPU parity of the streamed expert kernels (few token rows per expert): the lane layouts of a row (whole and padded, in
one wave and shared by four), items of one to eight rows and experts that take several, both pagers, fp8 and
bf16, against the oracle, and bit for bit against the resident run and (to four tokens) the device pager."""
import ctypes

import numpy as np
import pytest

import oracle
from parity import log, run_case
from paper_2606_21868_amd import wisp
from paper_2606_21868_amd.workloads import FP8, ROUTE_SIGMOID_GROUP, WORKLOADS

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BF16 = WORKLOADS["qwen3-30b-a3b-decode"]
F8 = BF16.with_(w_dtype=FP8, route=ROUTE_SIGMOID_GROUP, n_groups=4, topk_groups=2, has_shared=True)

CASES = {
    # up to four tokens: the device pager runs the same rows (checked bit for bit by run_case)
    "fp8 one token, both pagers": (F8.with_(L=2, T=1, d=7168, I=256, N=16, k=4), 5, 6),
    "fp8 four tokens, both pagers": (F8.with_(L=1, T=4, d=256, I=2048, N=16, k=4), 16, 3),
    "bf16 three tokens, both pagers": (BF16.with_(L=2, T=3, d=384, I=768, N=32, k=4), 12, 4),
    "bf16 two tokens, both pagers": (BF16.with_(L=1, T=2, d=2048, I=128, N=16, k=8), 16, 3),
    # rows padded to whole lanes' chunks (184 and 88 chunks), a shared expert of 15 rows (two items)
    "bf16 padded rows, shared": (BF16.with_(L=2, T=15, d=1472, I=704, N=12, k=3, has_shared=True), 5, 2),
    # rows shared by four waves, whole (1792 chunks) and padded (576 chunks: a last wave with few)
    "bf16 rows of four waves": (BF16.with_(L=1, T=5, d=4608, I=14336, N=4, k=2), 4, 1),
    # every lane layout that is not above: 8 x 16 lanes, 5 and 8 chunks
    "bf16 short rows": (BF16.with_(L=1, T=9, d=128, I=320, N=24, k=6), 7, 2),
    "bf16 wide rows": (BF16.with_(L=1, T=6, d=4096, I=2560, N=8, k=2), 4, 1),
    # fp8 with padded rows
    "fp8 padded rows": (F8.with_(L=1, T=7, d=2944 - 256, I=768, N=16, k=4), 8, 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_streamed_rows(name):
    wl, cap, steps = CASES[name]
    run_case(wl, cap, steps, check_all_outputs=True, expect_grouped=False)


# token batches below and at the line of five mean rows, with experts of more than eight rows; a batch just above it
# takes the grouped GEMMs.  More items than a launch takes: 230 experts.
@pytest.mark.parametrize("T,N,k,d,I,shared", [(16, 8, 2, 256, 128, False), (40, 16, 2, 256, 256, False),
                                              (41, 16, 2, 256, 256, False), (33, 12, 1, 320, 192, True),
                                              (120, 230, 8, 256, 128, False)])
def test_streamed_token_batches(T, N, k, d, I, shared):
    wl = WORKLOADS["qwen3-30b-a3b-prefill"].with_(L=1, T=T, N=N, k=k, d=d, I=I, has_shared=shared)
    run_case(wl, max(1, N // 3), 1, check_all_outputs=True, expect_grouped=True)


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
