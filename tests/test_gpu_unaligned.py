"""Rows that start anywhere: every kernel reads its rows with 16-byte loads whatever the base address
and the row stride, so the same values at any offset and stride give the same bits (the aligned layout
is compared with the oracle in the other files).  The widths sit around a chunk of 1,024 entries."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N, M = 3, 2


def shifted(rows, offset, pad, fill):
    """`rows` at `offset` elements into a buffer, with row stride width + pad; what lies between holds `fill`."""
    n, v = rows.shape
    buf = torch.full((offset + n * (v + pad) + 16,), fill, dtype=rows.dtype, device=rows.device)
    out = buf[offset:offset + n * (v + pad)].view(n, v + pad)
    out[:, :v] = rows
    return out


@pytest.mark.parametrize("offset,pad", [(1, 0), (2, 1), (3, 2), (5, 3)])
@pytest.mark.parametrize("v", [1023, 1024, 1025, 3075])
def test_same_bits_at_any_alignment(v, offset, pad):
    import paper_2510_15545_amd as tt

    g = torch.Generator(device="cuda").manual_seed(v * 16 + offset)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")  # noqa: E731
    rows = N * (M + 1)
    p = torch.softmax(3 * torch.randn((rows, v), generator=g, device="cuda"), 1)
    q = torch.softmax(3 * torch.randn((N * M, v), generator=g, device="cuda"), 1)
    logits = (3 * torch.randn((rows, v), generator=g, device="cuda")).bfloat16()
    ids = torch.randint(0, v, (N * M,), generator=g, device="cuda", dtype=torch.int32)
    off = (torch.arange(N + 1, device="cuda") * M).int()
    qs, ua, us, it = rnd(N * M) * 2e-3, rnd(N * M), rnd(N), 0.5 + rnd(N)
    order = torch.randperm(v, generator=g, device="cuda").int()
    d2t = torch.where(rnd(v) < 0.5, order, torch.full_like(order, -1))
    t2d = torch.full_like(d2t, -1)
    kept = torch.nonzero(d2t >= 0).flatten()
    t2d[d2t[kept].long()] = kept.int()

    def calls(place):
        P, Q, X = place(p, 7.0), place(q, 7.0), place(logits, 90.0)
        lse = torch.logsumexp(logits.float() * it.repeat_interleave(M + 1)[:, None], 1)
        res, dres = (torch.zeros((N, P.stride(0)), device="cuda") for _ in range(2))
        return (tt.verify(v, ids, off, qs, P, ua, us, M, out=(off.new_zeros(N), off.new_zeros(N), res)),
                tt.verify_dense(v, ids, off, Q, P, ua, us, M, out=(off.new_zeros(N), off.new_zeros(N), dres)),
                tt.verify_logits(v, ids, off, qs, X, it, ua, us, M),
                tt.verify_logits(v, ids, off, qs, X, it, ua, us, M, lse=lse),
                tt.verify_tli(d2t, t2d, ids, off, Q, P, ua, us, M),
                (tt.tli_proposal(d2t, t2d, Q, out=place(torch.zeros_like(p[:N * M]), 0.0)),))

    want, got = calls(lambda r, fill: r.contiguous()), calls(lambda r, fill: shifted(r, offset, pad, fill))
    torch.cuda.synchronize()
    for w, x in zip(want, got):
        for a, b in zip(w, x):
            assert torch.equal(a, b[..., :a.shape[-1]] if a.dim() == 2 else b)


def test_spread_calls_replay_in_a_graph():
    """The calls that take several kernels and scratch memory, captured once and replayed on new inputs in the same
    buffers, other work in between: every replay equals the eager call."""
    import paper_2510_15545_amd as tt

    n, m, v = 6, 5, 40000
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")  # noqa: E731
    off = (torch.arange(n + 1, device="cuda") * m).int()
    order = torch.randperm(v, generator=g, device="cuda").int()
    d2t, t2d = order, torch.empty_like(order)
    t2d[d2t.long()] = torch.arange(v, device="cuda").int()
    buf = dict(p=rnd(n * (m + 1), v), q=rnd(n * m, v), x=(3 * rnd(n * (m + 1), v)).bfloat16(), u=rnd(n * m), s=rnd(n),
               ids=torch.zeros(n * m, dtype=torch.int32, device="cuda"), it=0.5 + rnd(n), qs=rnd(n * m) * 1e-4)
    out = torch.zeros((n * m, v), device="cuda")

    def calls():
        lse = torch.zeros(n * (m + 1), device="cuda") + 12.0
        return (*tt.verify_logits(v, buf["ids"], off, buf["qs"], buf["x"], buf["it"], buf["u"], buf["s"], m),
                *tt.verify_logits(v, buf["ids"], off, buf["qs"], buf["x"], buf["it"], buf["u"], buf["s"], m, lse=lse),
                *tt.verify_tli(d2t, t2d, buf["ids"], off, buf["q"], buf["p"], buf["u"], buf["s"], m),
                tt.tli_proposal(d2t, t2d, buf["q"], out=out))

    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = calls()
    for _ in range(3):
        for k, t in buf.items():
            if k == "ids":
                t.copy_(torch.randint(0, v, t.shape, generator=g, device="cuda"))
            else:
                t.copy_((rnd(*t.shape) * (6 if k == "x" else 1e-4 if k == "qs" else 1) + (0.5 if k == "it" else 0)).to(t.dtype))
        graph.replay()
        replayed = [t.clone() for t in got]
        torch.cuda.synchronize()
        eager = calls()
        assert all(torch.equal(a, b) for a, b in zip(replayed, eager))
