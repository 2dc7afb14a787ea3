"""The calls that can do without a workspace (tt_verify_logits_ws, tt_verify_tli_ws): the caller's, none, one too
small, on a stream of the caller's, and while a capture is under way."""
import types

import pytest
import torch

pytestmark = pytest.mark.gpu

N, M, V = 6, 5, 40000


def inputs(seed=3):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")  # noqa: E731
    off = (torch.arange(N + 1, device="cuda") * M).int()
    order = torch.randperm(V, generator=g, device="cuda").int()
    t2d = torch.empty_like(order)
    t2d[order.long()] = torch.arange(V, device="cuda").int()
    ids = torch.randint(0, V, (N * M,), generator=g, device="cuda", dtype=torch.int32)
    return dict(off=off, d2t=order, t2d=t2d, ids=ids, p=rnd(N * (M + 1), V), q=rnd(N * M, V), u=rnd(N * M), s=rnd(N),
                x=(6 * rnd(N * (M + 1), V)).bfloat16(), it=0.5 + rnd(N), qs=rnd(N * M) * 1e-4,
                lse=torch.zeros(N * (M + 1), device="cuda") + 12.0)


def calls(i):
    """(call, workspace maker) of each entry point; a call takes keyword arguments."""
    import paper_2510_15545_amd as tt

    logits = lambda **kw: tt.verify_logits(V, i["ids"], i["off"], i["qs"], i["x"], i["it"], i["u"], i["s"], M, **kw)  # noqa: E731
    tli = lambda **kw: tt.verify_tli(i["d2t"], i["t2d"], i["ids"], i["off"], i["q"], i["p"], i["u"], i["s"], M, **kw)  # noqa: E731
    return [(logits, lambda: tt.verify_logits_workspace(N, V, M)),
            (lambda **kw: logits(lse=i["lse"], **kw), lambda: tt.verify_logits_workspace(N, V, M, lse=True)),
            (tli, lambda: tt.verify_tli_workspace(N, V))]


def fresh():
    return tuple(torch.full((N,), -7, dtype=torch.int32, device="cuda") for _ in range(2))


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def allocations():
    return torch.cuda.memory_stats()["allocation.all.allocated"]


def test_the_callers_workspace():
    import paper_2510_15545_amd as tt

    for call, make in calls(inputs()):
        want = call(workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
        ws, out = make(), fresh()
        assert ws.numel() > 0
        torch.cuda.synchronize()
        before = allocations()
        got = call(workspace=ws, out=out)
        assert allocations() == before  # nothing is allocated beside it
        assert same(want, got) and same(want, call())
        with pytest.raises(tt.TTError):
            call(workspace=ws[:-1])
        with pytest.raises(ValueError):
            call(workspace=ws.cpu())


def test_a_capture_allocates_nothing_beside_the_callers_tensors():
    """With out= given, a call under capture runs without scratch of its own: a capture begun outside torch would
    keep its address, but not the memory."""
    i = inputs()
    for k, (call, make) in enumerate(calls(i)):
        want, out = call(), fresh()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            before = allocations()
            call(out=out)
            assert allocations() == before, k
        for _ in range(3):
            for t in out:
                t.fill_(-7)
            graph.replay()
            assert same(want, out), k


def test_streams_of_the_callers():
    """torch's streams, and any object with a handle; the scratch is freed to the stream that used it."""
    i = inputs()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for call, _ in calls(i):
        want = call()
        torch.cuda.synchronize()
        for s in (side, types.SimpleNamespace(cuda_stream=side.cuda_stream)):
            out = fresh()
            torch.cuda.synchronize()
            call(out=out, stream=s)
            side.synchronize()
            assert same(want, out)
