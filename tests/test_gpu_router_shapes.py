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


def _route_run(T):
    run = wisp.DecodeRun(BASE.with_(T=T, N=24, d=256), device=0, steps=1)
    run.generate()
    xs = [torch.randn(T, 256, device=run.dev, generator=torch.Generator(run.dev).manual_seed(i)).to(torch.bfloat16) for i in range(6)]
    out = lambda: (torch.zeros((T, 2), dtype=torch.int32, device=run.dev), torch.zeros((T, 2), device=run.dev))

    def eager(x):
        idx, w = out()
        run.ctx.route_topk(0, x, T, idx, w, np.zeros(T * 2, np.int32), run.stream)
        run.stream.synchronize()
        return idx, w
    return run, xs, out, eager


@pytest.mark.parametrize("T", [1, 4, 6, 8, 9])
@pytest.mark.parametrize("noalloc", [False, True])
def test_captured_routing_replays(T, noalloc):
    # a graph's replays repeat the arguments of its launches, the one-launch router's tag among them
    log(f"[case] captured routing T={T} {'noalloc' if noalloc else 'context'}")
    run, xs, out, eager = _route_run(T)
    try:
        want = [eager(x) for x in xs]
        x, (idx, w) = xs[0].clone(), out()

        def call():
            if noalloc:
                wisp.route_topk_noalloc(run.wr_dev[0], x, wisp.BF16, T, 24, 256, 2, BASE.route, 1, 1, idx, w, run.stream)
            else:
                run.ctx.route_topk(0, x, T, idx, w, None, run.stream)
        with torch.cuda.stream(run.stream):
            call()   # (the context-free scratch clears its words once, outside the graph)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=run.stream):
            call()
        for i in (1, 2, 3, 4, 5, 0, 1, 2, 5, 4):
            x.copy_(xs[i])
            idx.fill_(-1)
            torch.cuda.synchronize()
            with torch.cuda.stream(run.stream):
                g.replay()
            torch.cuda.synchronize()
            assert torch.equal(idx, want[i][0]) and torch.equal(w, want[i][1]), i
            if i == 3:   # its own work between replays (it leaves words of another tag, so not between all of them)
                eager(xs[4])
    finally:
        run.close()


@pytest.mark.parametrize("T", [2, 8])
def test_routing_on_two_streams_in_turn(T):
    # calls that wait for nothing, on two streams of one context, which share its tagged words
    log(f"[case] routing on two streams T={T}")
    run, xs, out, eager = _route_run(T)
    try:
        want = [eager(x) for x in xs]
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        got = [out() for _ in range(24)]
        torch.cuda.synchronize()
        for i, (idx, w) in enumerate(got):
            run.ctx.route_topk(0, xs[i % 6], T, idx, w, None, streams[i // 3 % 2])
        torch.cuda.synchronize()
        for i, (idx, w) in enumerate(got):
            assert torch.equal(idx, want[i % 6][0]) and torch.equal(w, want[i % 6][1]), i
    finally:
        run.close()
