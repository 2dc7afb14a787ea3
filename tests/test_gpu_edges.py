"""GPU edge cases, each compared with the oracle (or with the documented sentinel)."""
import numpy as np
import pytest

from gpu_util import compare_align, compare_verify, gpu_run, oracle_run, to_dev
from paper_2510_15545_amd import synth

pytestmark = pytest.mark.gpu


def vocab_of(tokens):
    tokens = list(tokens)
    off = np.zeros(len(tokens) + 1, np.int32)
    off[1:] = np.cumsum([len(t) for t in tokens])
    data = np.frombuffer(b"".join(tokens), np.uint8).copy()
    return synth.Vocab(tokens, {t: i for i, t in enumerate(tokens)}, data, off,
                       max([len(t) for t in tokens]))


def workload(vd, vt, pairs, v_d, v_t, w=8, seed=0, probs=True):
    def csr(lists):
        off = np.zeros(len(lists) + 1, np.int32)
        off[1:] = np.cumsum([len(l) for l in lists])
        return np.array([x for l in lists for x in l], np.int32), off

    di, do = csr([p[0] for p in pairs])
    ti, to = csr([p[1] for p in pairs])
    spec = synth.Spec(0, "edge", len(pairs), 0, v_d, v_t, b"", 64, None, w)
    wl = synth.Workload(spec, vd, vt, di, do, ti, to, w, v_d=v_d, v_t=v_t, verify_ids=ti)
    if probs:
        rng = np.random.default_rng(seed)
        n = len(pairs)

        def rows(k, width):
            x = rng.standard_normal((k, width)).astype(np.float32) * np.float32(2)
            e = np.exp(x - x.max(axis=1, keepdims=True)).astype(np.float32)
            return (e / e.sum(axis=1, keepdims=True, dtype=np.float32)).astype(np.float32)

        wl.draft_probs = rows(int(do[-1]), v_d)
        wl.target_probs = rows(int(to[-1]) + n, v_t)
        wl.u_accept = (rng.integers(0, 1 << 24, int(to[-1])) * 2.0**-24).astype(np.float32)
        wl.u_sample = (rng.integers(0, 1 << 24, n) * 2.0**-24).astype(np.float32)
    return wl


def random_tokens(rng, n, lo, hi, alphabet=b"abcdefgh"):
    out = set()
    alpha = np.frombuffer(alphabet, np.uint8)
    while len(out) < n:
        ln = int(rng.integers(lo, hi + 1))
        out.add(alpha[rng.integers(0, len(alpha), ln)].tobytes())
    return sorted(out)


@pytest.mark.parametrize("maxlen", [8, 16, 32, 64])
def test_token_slot_widths(maxlen):
    """Every token-width instantiation (8/16/32/64-byte slots) against the oracle."""
    print(f"[case] token slots maxlen={maxlen}", flush=True)
    rng = np.random.default_rng(maxlen)
    toks_d = random_tokens(rng, 300, 1, maxlen, bytes(range(0x20, 0x7F)) + b"\x00\xc3\xa9")
    toks_t = random_tokens(rng, 400, 1, maxlen, bytes(range(0x20, 0x7F)) + b"\x00\xc3\xa9")
    vd, vt = vocab_of(toks_d), vocab_of(toks_t)
    pairs = [(list(rng.integers(0, len(toks_d), rng.integers(1, 40))),
              list(rng.integers(0, len(toks_t), rng.integers(1, 40)))) for _ in range(40)]
    wl = workload(vd, vt, pairs, len(toks_d), len(toks_t))
    for w in (8, -1, 3):
        o = oracle_run(wl, w=w)
        g = gpu_run(wl, w=w)  # row-scan kernel
        compare_align(wl, g, o)
        compare_verify(g, o)
        compare_align(wl, gpu_run(wl, w=w, bounds=(65, 65)), o)  # strip kernel


def test_strips_longer_than_a_wave():
    """K and M well above 64 rows, every w in the paper's sweep (strip boundaries, band widening)."""
    rng = np.random.default_rng(5)
    toks = random_tokens(rng, 200, 1, 4)
    v = vocab_of(toks)
    pairs = []
    # band widths up to and past the widest precomputed band (512 cells per row): 64-row
    # strips whose band shifts one column per row span up to W + 126 sweep steps
    for k, m in ((65, 64), (64, 65), (130, 129), (200, 60), (60, 200), (128, 128), (1, 300), (300, 1),
                 (150, 100), (100, 150), (200, 210), (300, 520), (260, 520), (520, 300)):
        pairs.append((list(rng.integers(0, len(toks), k)), list(rng.integers(0, len(toks), m))))
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    for w in (4, 8, 16, -1, 0, 40, 70):
        print(f"[case] strips w={w}", flush=True)
        compare_align(wl, gpu_run(wl, w=w), oracle_run(wl, w=w))


def test_band_rows_wider_than_a_wave_of_code_words():
    """Band rows of more than 64 code words (W > 1008 cells): the backtrack reads code words
    from the workspace instead of staging strips in LDS, and a run may cross many words."""
    rng = np.random.default_rng(11)
    toks = random_tokens(rng, 120, 1, 4)
    v = vocab_of(toks)
    pairs = []
    for k, m in ((100, 1100), (1100, 100), (1030, 1050), (700, 1100), (1, 1100), (1100, 1)):
        pairs.append((list(rng.integers(0, len(toks), k)), list(rng.integers(0, len(toks), m))))
    # long runs of one repeated draft token make the path cross whole code words in one row
    pairs.append(([3] * 40, list(rng.integers(0, len(toks), 1100))))
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    for w in (8, -1):
        print(f"[case] wide rows w={w}", flush=True)
        compare_align(wl, gpu_run(wl, w=w), oracle_run(wl, w=w))


@pytest.mark.parametrize("kernel", ["rows", "strips"])
def test_short_pair_extremes(kernel):
    """Pairs at the row-scan kernel's limits (K, M in {1, 63, 64}), through both alignment
    kernels: bounds of 64 select the row-scan kernel, a bound of 65 the strip kernel."""
    rng = np.random.default_rng(11)
    toks = random_tokens(rng, 120, 1, 6)
    v = vocab_of(toks)
    shapes = ((64, 64), (1, 64), (64, 1), (1, 1), (63, 64), (64, 63), (64, 30), (30, 64), (2, 64), (64, 2))
    pairs = [(list(rng.integers(0, len(toks), k)), list(rng.integers(0, len(toks), m))) for k, m in shapes]
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    bounds = (64, 64) if kernel == "rows" else (65, 64)
    for w in (0, 1, 4, 8, -1, 70):
        print(f"[case] short pair extremes kernel={kernel} w={w}", flush=True)
        compare_align(wl, gpu_run(wl, w=w, bounds=bounds), oracle_run(wl, w=w))


@pytest.mark.parametrize("c", [2, 3, 5])
def test_strip_kernel_on_benchmark_shapes(c):
    """The strip kernel stays bit-exact on the short pairs the row-scan kernel normally takes."""
    from paper_2510_15545_amd import synth

    print(f"[case] strip kernel on workload {c}", flush=True)
    wl = synth.make(c, n_streams=16)
    for w in (8, -1):
        g = gpu_run(wl, w=w, bounds=(max(65, wl.max_k), max(65, wl.max_m)))
        compare_align(wl, g, oracle_run(wl, w=w))


def test_sentinel_pairs_and_streams():
    rng = np.random.default_rng(6)
    toks = random_tokens(rng, 50, 1, 5)
    v = vocab_of(toks)
    pairs = [([1, 2, 3], [4, 5]), ([1, 999], [3]), ([2, 3], [4, -1]), ([5], [6, 7, 8])]
    wl = workload(v, v, pairs, len(toks), len(toks))
    wl.verify_ids = wl.target_ids.copy()
    wl.verify_ids[wl.target_off[2] + 1] = 10**6  # out of range for verify as well
    g, o = gpu_run(wl), oracle_run(wl)
    compare_align(wl, g, o)
    assert list(g["cost"][1:3]) == [-1, -1] and list(g["map"][wl.target_off[1]:wl.target_off[3]]) == [-1] * 3
    compare_verify(g, o)
    assert int(g["n_accepted"][2]) == -1 and int(g["out_token"][2]) == -1


def test_bounds_smaller_than_pairs_give_sentinels():
    import paper_2510_15545_amd as tt

    rng = np.random.default_rng(7)
    toks = random_tokens(rng, 50, 1, 5)
    v = vocab_of(toks)
    pairs = [([1, 2, 3], [4, 5]), ([1, 2, 3, 4, 5, 6], [3]), ([2], [4, 5, 6, 7, 8, 9])]
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    from gpu_util import upload

    d = upload(wl)
    cost, plen, path, mp = tt.align(d["vd"], d["vt"], d["draft_ids"], d["draft_off"], d["target_ids"],
                                    d["target_off"], 8, 4, 4)
    cost = cost.cpu().numpy()
    assert cost[0] >= 0 and cost[1] == -1 and cost[2] == -1
    assert list(mp.cpu().numpy()[wl.target_off[2]:]) == [-1] * 6


def test_verify_edge_values():
    """M = 0 streams, q = 0 / NaN, u at the ends of [0,1), a zero-mass residual, rows not 16-B aligned."""
    import torch
    import oracle
    import paper_2510_15545_amd as tt

    V, ld = 3001, 3003  # ragged tail, ld % 4 != 0 -> scalar loads
    rng = np.random.default_rng(8)
    n = 7
    Ms = [0, 1, 2, 3, 1, 2, 1]
    off = np.zeros(n + 1, np.int32)
    off[1:] = np.cumsum(Ms)
    ids = rng.integers(0, V, int(off[-1])).astype(np.int32)
    rows = rng.random((int(off[-1]) + n, ld)).astype(np.float32)
    rows /= rows[:, :V].sum(axis=1, keepdims=True, dtype=np.float32)
    q = rng.random(int(off[-1])).astype(np.float32)
    ua = (rng.integers(0, 1 << 24, int(off[-1])) * 2.0**-24).astype(np.float32)
    us = (rng.integers(0, 1 << 24, n) * 2.0**-24).astype(np.float32)
    q[off[1]] = 0.0             # stream 1: q = 0 -> accepted
    q[off[2]] = np.nan          # stream 2: NaN proposal -> rejected
    us[3] = 0.0
    us[4] = np.float32(1 - 2**-24)
    # stream 5: the residual is empty (all mass on the rejected proposal, q > 1)
    r5 = off[5] + 5
    rows[r5, :] = 0.0
    rows[r5, ids[off[5]]] = 1.0
    q[off[5]] = 2.0
    ua[off[5]] = 0.9
    # stream 6: NaN and negative entries in the bonus row, q tiny -> accepted
    q[off[6]] = 1e-30
    rows[off[6] + 6 + 1, 5] = np.nan
    rows[off[6] + 6 + 1, 6] = -0.5
    rows_c = np.ascontiguousarray(rows)
    o_nacc, o_tok, o_res, _ = oracle.verify(V, ids, off, q, rows_c, ua, us, residual=True)
    dev = {k: to_dev(v) for k, v in dict(ids=ids, off=off, q=q, ua=ua, us=us).items()}
    P = to_dev(rows_c)
    nacc, tok, res = tt.verify(V, dev["ids"], dev["off"], dev["q"], P, dev["ua"], dev["us"], 3, residual=True)
    torch.cuda.synchronize()
    assert np.array_equal(nacc.cpu().numpy(), o_nacc)
    assert np.array_equal(tok.cpu().numpy(), o_tok)
    r = res.cpu().numpy()[:, :V]
    ro = o_res[:, :V]
    assert np.all(np.abs(r.astype(np.float64) - ro) <= 1e-6 * np.abs(ro))
    assert int(o_tok[5]) == int(ids[off[5]])  # zero-mass fallback = first argmax


def test_empty_batch_and_argument_errors():
    import torch
    import paper_2510_15545_amd as tt

    e = torch.zeros(1, dtype=torch.int32, device="cuda")
    off = torch.zeros(1, dtype=torch.int32, device="cuda")
    P = torch.zeros((1, 8), dtype=torch.float32, device="cuda")
    f = torch.zeros(1, dtype=torch.float32, device="cuda")
    nacc, tok, _ = tt.verify(8, e, off, f, P, f, f, 0)
    assert nacc.numel() == 0 and tok.numel() == 0
    with pytest.raises(tt.TTError):
        tt.verify(8, e, torch.zeros(2, dtype=torch.int32, device="cuda"), f, P, f, f, -1)


@pytest.mark.parametrize("w", [-1, 0, 3, 8])
def test_strip_walk_segment_and_group_boundaries(w):
    """Pairs whose row counts sit on and around the 32-row segments and 64-row strips of the
    strip kernel's backtrack (segments walked in parallel from guessed columns, then corrected),
    with several band widths, some pairs far off the diagonal: bit-exact against the oracle."""
    print(f"[case] strip walk boundaries w={w}", flush=True)
    rng = np.random.default_rng(100 + w)
    toks = random_tokens(rng, 120, 1, 6, alphabet=b"abcdefgh")
    v = vocab_of(toks)
    ks = [31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 200, 257, 300]
    pairs = []
    for k in ks:
        for m in (max(1, k // 3), k, k + 37, 2 * k):
            d = list(rng.integers(0, len(toks), k))
            # targets that share long stretches with the drafts (paths near the diagonal) or not
            t = (d[:m] + list(rng.integers(0, len(toks), max(0, m - k)))) if rng.random() < 0.5 else \
                list(rng.integers(0, len(toks), m))
            pairs.append((d, t))
    wl = workload(v, v, pairs, len(toks), len(toks), w=w, probs=False)
    g = gpu_run(wl, w=w)
    compare_align(wl, g, oracle_run(wl, w=w))


@pytest.mark.parametrize("n,V,dense", [(256, 300_000, False), (3, 9_000_000, False), (256, 300_000, True)])
def test_large_vocabularies(n, V, dense):
    """Rows past 256 chunks (the sampler's chunk sums no longer fit four per lane) on the
    one-workgroup-per-stream path, and rows past 8M floats (over the row path's LDS) on the
    split path; one-hot and dense proposals, bit-exact against the oracle."""
    print(f"[case] large vocabulary n={n} V={V} dense={dense}", flush=True)
    verify_case(n, V, dense)


@pytest.mark.parametrize("V", [640, 12_000, 30_000, 50_000, 100_000])
@pytest.mark.parametrize("dense", [False, True])
def test_row_path_workgroup_sizes(V, dense):
    """The one-workgroup-per-stream path sizes its workgroup from the row (about eight 1024-float
    chunks per wave): 64, 128, 256, 512 and 1024 threads for these widths."""
    print(f"[case] row path n=256 V={V} dense={dense}", flush=True)
    verify_case(256, V, dense)


def verify_case(n, V, dense):
    """Random rows of width V for n streams with 0-2 proposals each; GPU outputs against the
    oracle, bit for bit (one-hot proposals through tt_verify, dense through tt_verify_dense)."""
    import torch

    import oracle
    import paper_2510_15545_amd as tt

    rng = np.random.default_rng(V + n)
    Ms = rng.integers(0, 3, n)
    off = np.zeros(n + 1, np.int32)
    off[1:] = np.cumsum(Ms)
    nt = int(off[-1])
    ids = rng.integers(0, V, nt).astype(np.int32)
    rows = rng.random((nt + n, V), dtype=np.float32)
    rows /= rows.sum(axis=1, keepdims=True, dtype=np.float32)
    ids[::3] = np.argmax(rows[(off[:-1] + np.arange(n))[np.repeat(np.arange(n), Ms)][::3]], axis=1)  # likely accepts
    ua = (rng.integers(0, 1 << 24, nt) * 2.0**-24).astype(np.float32)
    us = (rng.integers(0, 1 << 24, n) * 2.0**-24).astype(np.float32)
    us[0] = np.float32(1 - 2**-24)
    P = to_dev(rows)
    if dense:
        qrows = rng.random((max(1, nt), V), dtype=np.float32)
        qrows /= qrows.sum(axis=1, keepdims=True, dtype=np.float32)
        o_nacc, o_tok, _, _ = oracle.sd_verify(V, ids, off, qrows[:nt], rows, ua, us)
        nacc, tok, _ = tt.verify_dense(V, to_dev(ids), to_dev(off), to_dev(qrows), P, to_dev(ua), to_dev(us), 2)
    else:
        q = rng.random(nt).astype(np.float32) * np.float32(1e-5)
        o_nacc, o_tok, _, _ = oracle.verify(V, ids, off, q, rows, ua, us)
        nacc, tok, _ = tt.verify(V, to_dev(ids), to_dev(off), to_dev(q), P, to_dev(ua), to_dev(us), 2)
    torch.cuda.synchronize()
    assert np.array_equal(nacc.cpu().numpy(), o_nacc)
    assert np.array_equal(tok.cpu().numpy(), o_tok)
    assert 0 < (o_nacc < Ms).sum() or n < 8


@pytest.mark.parametrize("maxlen,n", [(8, 5), (8, 257), (16, 5), (16, 256), (16, 257)])
def test_distance_forms_of_the_strip_kernel(maxlen, n):
    """Every form of the token distance (short drafts, short targets, neither), mixed and alone, empty tokens among
    them, in strips of one chunk (M = 1) and of several, with and without the match tables and the ranking."""
    rng = np.random.default_rng(100 * maxlen + n)
    alphabet = b"ab\x00\xff"
    kinds = [random_tokens(rng, 10, 1, 2, alphabet), random_tokens(rng, 40, 3, 4, alphabet),
             random_tokens(rng, 60, 5, maxlen, alphabet)]
    toks = [b""] + [t for k in kinds for t in k]
    first = np.cumsum([0, 1] + [len(k) for k in kinds])  # ids of the empty token and of each kind
    v = vocab_of(toks)
    choose = {"empty": (0, 1), "short": (1, 2), "four": (1, 3), "long": (3, 4), "any": (0, 4)}

    def ids(kind, count):
        a, b = choose[kind]
        return list(rng.integers(first[a], first[b], count))

    mixes = [("short", "four"), ("short", "any"), ("long", "short"), ("long", "four"), ("any", "short"), ("any", "any"),
             ("long", "long"), ("empty", "short"), ("short", "empty")]
    sizes = [(130, 40), (65, 1), (70, 150), (3, 80), (64, 64), (129, 2)]
    pairs = [(ids(mixes[p % len(mixes)][0], sizes[p // 2 % len(sizes)][0]), ids(mixes[p % len(mixes)][1], sizes[p // 2 % len(sizes)][1]))
             for p in range(n)]
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    for w in (8, -1):
        compare_align(wl, gpu_run(wl, w=w), oracle_run(wl, w=w))


@pytest.mark.parametrize("n_bins", [1, 3, 255, 256, 257, 1024, 8191, 8192])
def test_delta_quantile_sizes(n_bins):
    """One bin to the most, against the definition in Python integers."""
    import paper_2510_15545_amd as tt

    rng = np.random.default_rng(n_bins)
    for h in (rng.integers(0, 2 ** 31 - 1, n_bins), rng.integers(0, 2, n_bins), np.eye(1, n_bins, n_bins - 1)[0], np.zeros(n_bins)):
        h = h.astype(np.int32)
        cum = np.cumsum(h.astype(np.int64))
        for num, den in ((9, 10), (0, 1), (1, 1), (65535, 65536)):
            want = 0 if cum[-1] == 0 else next(d for d in range(n_bins) if int(cum[d]) * den >= num * int(cum[-1]))
            assert tt.w_at_quantile(to_dev(h), num, den) == want, (n_bins, num, den)


@pytest.mark.parametrize("K,M,short_of", [(4, 70, 0), (4, 70, 1), (67, 90, 0), (67, 90, 1), (130, 65, 0), (130, 65, 1)])
def test_match_tables_by_the_share_of_long_drafts(K, M, short_of):
    """Pairs with a quarter of their draft tokens longer than six bytes, and with one less: distances from match tables
    and from gathered masks, pairs of both kinds in one batch."""
    rng = np.random.default_rng(K + M + short_of)
    alphabet = b"ab\x00\xff"
    short, long_ = random_tokens(rng, 40, 1, 6, alphabet), random_tokens(rng, 60, 7, 16, alphabet)
    toks = short + long_
    v = vocab_of(toks)
    pairs = []
    for p in range(9):
        n_long = -(-K // 4) - short_of * (p % 2)
        d = np.concatenate([rng.integers(40, 100, n_long), rng.integers(0, 40, K - n_long)])
        pairs.append((list(rng.permutation(d)), list(rng.integers(0, (100, 40, 100)[p % 3], M))))
    wl = workload(v, v, pairs, len(toks), len(toks), probs=False)
    for w in (8, -1):
        compare_align(wl, gpu_run(wl, w=w, bounds=(max(K, 70), M)), oracle_run(wl, w=w))


@pytest.mark.parametrize("V", [1, 2, 3, 4, 5, 1023, 1027, 2047, 2048, 2049, 2051, 3071, 3074, 4095, 6147])
@pytest.mark.parametrize("dense", [False, True])
def test_residual_rows_of_any_width(V, dense):
    """Whole spans of 2,048 entries, ragged ends of 16-byte groups and of one to three entries, a row without mass."""
    import torch

    import paper_2510_15545_amd as tt

    n, M = 5, 2
    g = torch.Generator(device="cuda").manual_seed(V)
    p = torch.rand((n * (M + 1), V), generator=g, device="cuda") / V
    q = torch.rand((n * M, V), generator=g, device="cuda") / V
    p[3], q[2] = 0.0, 1.0  # stream 1 stops at its first row, and has no mass there
    ids = torch.randint(0, V, (n * M,), generator=g, device="cuda", dtype=torch.int32)
    off = (torch.arange(n + 1, device="cuda") * M).int()
    ua, us = torch.full((n * M,), 0.9, device="cuda"), torch.rand(n, generator=g, device="cuda")
    if dense:
        nacc, tok, res = tt.verify_dense(V, ids, off, q, p, ua, us, M, residual=True)
    else:
        one = torch.rand(n * M, generator=g, device="cuda")
        nacc, tok, res = tt.verify(V, ids, off, one, p, ua, us, M, residual=True)
    torch.cuda.synchronize()
    for b in range(n):
        r = int(nacc[b])
        R = p[b * (M + 1) + r].clone()
        if r < M and dense:
            R -= q[b * M + r]
        elif r < M:
            R[ids[b * M + r]] -= one[b * M + r]
        R = R.clamp(0, 1)
        Z = sum(int(float(x) * 2.0 ** 62) for x in R.tolist())
        want = R / torch.tensor(Z * 2.0 ** -62, dtype=torch.float32, device="cuda") if Z else \
            torch.nn.functional.one_hot(tok[b].long(), V).float()
        # (Z rounds to fp32 here through a double: within one step, and the quotient within another)
        assert torch.allclose(res[b, :V], want, rtol=3 * 2.0 ** -24, atol=0), (b, r)


def test_residual_rows_in_several_launches():
    """More spans than a launch takes: every stream's row equals that of the stream in a small batch."""
    import torch

    import paper_2510_15545_amd as tt

    n, V = 4100, 131073  # 65 spans a row, 266,500 in all
    p = torch.rand((n, V), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    off = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    none_i, none_f = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
    us = torch.rand(n, device="cuda")
    _, tok, res = tt.verify(V, none_i, off, none_f, p, none_f, us, 0, residual=True)
    for a in (0, 2040, n - 8):
        _, t, r = tt.verify(V, none_i, off[:9], none_f, p[a:a + 8], none_f, us[a:a + 8].clone(), 0, residual=True)
        assert torch.equal(tok[a:a + 8], t) and torch.equal(res[a:a + 8], r)
