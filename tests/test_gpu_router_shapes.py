"""Router and top-k over the sizes where its launches change: up to eight tokens in one launch (a selecting workgroup
per token, or per four when there are fewer router rows than tokens), token batches over column slices
with remainders, row groups with rows past N.  Ids and gates against the oracle; one launch against two, bit for bit."""
import numpy as np
import pytest

from parity import check_gates, check_routing, log, oracle_routing, routing_bound
from paper_2606_21868_amd import wisp
from paper_2606_21868_amd.workloads import F32, WORKLOADS

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

BASE = WORKLOADS["qwen3-30b-a3b-prefill"].with_(L=1, I=64, k=2)


@pytest.mark.parametrize("T,N,d,x32", [(5, 24, 256, False), (8, 2, 256, False), (8, 24, 1088, True), (9, 60, 1472, False),
                                       (17, 3, 320, False), (33, 130, 704, True), (1040, 72, 640, False),
                                       (1100, 130, 704, False), (1000, 250, 704, True)])
def test_routing_against_oracle(T, N, d, x32):
    wl = BASE.with_(T=T, N=N, d=d, **(dict(w_dtype=F32, x_dtype=F32) if x32 else {}))
    log(f"[case] routing T={T} N={N} d={d} {'f32' if x32 else 'bf16'}")
    run = wisp.DecodeRun(wl, device=0, steps=1)
    try:
        run.generate()
        got = []
        for fusion in (1, 0):
            run.ctx.set_fusion(fusion)
            idx = torch.zeros((T, wl.k), dtype=torch.int32, device=run.dev)
            w = torch.zeros((T, wl.k), dtype=torch.float32, device=run.dev)
            ids = np.zeros(T * wl.k, np.int32)
            run.ctx.route_topk(0, run.x_dev[0, 0], T, idx, w, ids, run.stream)
            run.stream.synchronize()
            assert np.array_equal(ids, idx.cpu().numpy().ravel())
            got.append((idx.cpu().numpy()[None, None], w.cpu().numpy()[None, None]))
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1].view(np.uint32), got[1][1].view(np.uint32))
        ora_idx, ora_g, margin, gmargin, scores = oracle_routing(run, 1)
        exempt, reordered = check_routing(wl, got[0][0], ora_idx, margin, gmargin, scores)
        assert len(exempt) + len(reordered) <= routing_bound(1, wl)
        check_gates(run, got[0][0], got[0][1], ora_idx, ora_g, exempt)
    finally:
        run.close()
