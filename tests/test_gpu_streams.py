"""One context on several main streams: the memory in which launches share
tiles serves one stream at a time, so calls that overlap give the same bits as
calls one after the other."""
import pytest
import torch

from tests.gpu_util import bits, log

pytestmark = pytest.mark.gpu


def _calls(hcms, ctx, S, H, n, mode):
    """n independent calls (inputs, workspaces, output), each with the result
    of one head at a time."""
    scale = 128 ** -0.5
    calls = []
    for i in range(n):
        g = torch.Generator().manual_seed(100 * S + i)
        q, k, v = (torch.randn(S, H, 128, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
        hm = [x.permute(1, 0, 2).contiguous() for x in (q, k, v)]
        want = torch.cat([hcms.attention(*(x[h:h + 1].contiguous() for x in hm), scale) for h in range(H)])
        ws = [torch.empty(H, S, 128, dtype=torch.bfloat16, device="cuda") for _ in range(4)]
        out = torch.empty_like(q)

        def run(q=q, k=k, v=v, ws=ws, out=out):
            ctx.forward(q, k, v, 1, scale, (H,), mode=mode, out=out, workspaces=ws)
        calls.append((run, out, want.permute(1, 0, 2).contiguous()))
    torch.cuda.synchronize()
    return calls


@pytest.mark.parametrize("S,H,n", [(7800, 5, 2), (4096, 5, 2), (4000, 2, 5)])   # 155 tiles, 80, 32
def test_calls_on_several_streams_keep_their_results(hcms, S, H, n):
    log(f"[streams] S={S} H={H} streams={n}")
    ctx = hcms.Context()
    calls = _calls(hcms, ctx, S, H, n, hcms.MODE_SERIAL)
    streams = [torch.cuda.Stream() for _ in range(n)]
    for rep in range(6):
        for _, out, _ in calls:
            out.zero_()
        torch.cuda.synchronize()
        for i in range(2 * n):
            with torch.cuda.stream(streams[i % n]):
                calls[i % n][0]()
        torch.cuda.synchronize()
        for i, (_, out, want) in enumerate(calls):
            assert torch.equal(bits(out), bits(want)), (rep, i)
    ctx.close()


def test_replays_beside_calls_on_another_stream(hcms):
    """Warmed up and used on one stream, captured on another: replays overlap
    the calls on the first."""
    S, H = 7800, 5
    log(f"[streams] replays S={S} H={H}")
    ctx = hcms.Context()
    (run, out, want), (replayed, out_g, want_g) = _calls(hcms, ctx, S, H, 2, hcms.MODE_SERIAL)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        run()
        replayed()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=b):
        replayed()
    for rep in range(6):
        out.zero_()
        out_g.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(b):
            graph.replay()
        with torch.cuda.stream(a):
            run()
            run()
        torch.cuda.synchronize()
        assert torch.equal(bits(out), bits(want)), rep
        assert torch.equal(bits(out_g), bits(want_g)), rep
    ctx.close()
