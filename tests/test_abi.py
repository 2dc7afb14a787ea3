"""The C-ABI library: loads on a host without a GPU, exports every declared symbol,
and rejects host-visible argument errors before touching the device."""
import ctypes
import os
import re
import subprocess
import sys
import types

import pytest

import paper_2510_15545_amd as tt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "tt.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tt_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert {"tt_align", "tt_transfer", "tt_verify", "tt_status_string"} <= set(names)
    lib = ctypes.CDLL(tt.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n


def test_status_strings_and_version():
    L = tt.lib()
    for code in (0, -1, -2, -3, -4, 7):
        assert L.tt_status_string(code)
    assert L.tt_version() >= 100


def test_workspace_sizes_are_host_computed():
    L = tt.lib()
    n = ctypes.c_size_t(0)
    assert L.tt_verify_workspace_size(256, 151936, ctypes.byref(n)) == 0
    # Q62 mass + gamma per stream, and one Q62 sum per 1024-float chunk per stream
    assert n.value >= 256 * (8 + 4) + 256 * 149 * 8
    assert L.tt_verify_workspace_size(-1, 10, ctypes.byref(n)) == tt.TT_EINVAL
    assert L.tt_align_workspace_size(256, 8, 64, 8, 8, ctypes.byref(n)) == 0 and n.value == 0
    def strip_ws(pairs, words_per_pair):  # 2-bit codes, then the dispatch order (one int per pair)
        return ((4 * pairs * words_per_pair + 255) // 256) * 256 + 4 * pairs

    assert L.tt_align_workspace_size(1024, 512, 512, 8, 8, ctypes.byref(n)) == 0
    assert n.value == strip_ws(1024, 512 * 33)  # 2-bit codes for a 512-wide band row starting mid-word
    assert L.tt_align_workspace_size(8, 4096, 4096, -1, 8, ctypes.byref(n)) == 0
    assert n.value == strip_ws(8, 4096 * 257)
    # short pairs in a batch with one long target still take the strip kernel's workspace
    assert L.tt_align_workspace_size(4, 8, 100, 8, 8, ctypes.byref(n)) == 0 and n.value == strip_ws(4, 8 * 8)
    # one pair needs no dispatch order; above 2,048 pairs the order is not sorted
    assert L.tt_align_workspace_size(1, 8, 100, 8, 8, ctypes.byref(n)) == 0 and n.value == 8 * 8 * 4
    assert L.tt_align_workspace_size(2049, 8, 100, 8, 8, ctypes.byref(n)) == 0 and n.value == 2049 * 8 * 8 * 4
    assert L.tt_align_workspace_size(2048, 8, 100, 8, 8, ctypes.byref(n)) == 0 and n.value == strip_ws(2048, 64)
    assert L.tt_align_workspace_size(8, 4096, 4096, -1, 16, ctypes.byref(n)) == tt.TT_EUNSUPPORTED
    assert L.tt_align_workspace_size(8, 16, 16, 8, 65, ctypes.byref(n)) == tt.TT_EUNSUPPORTED
    # tt_step shares one workspace between its stages: the larger of the two
    a, v = ctypes.c_size_t(0), ctypes.c_size_t(0)
    for args in ((256, 151936, 8, 30, 8, 8), (1024, 151936, 512, 512, 8, 8), (4, 32000, 100, 100, -1, 16)):
        assert L.tt_step_workspace_size(*args, ctypes.byref(n)) == 0
        assert L.tt_align_workspace_size(args[0], args[2], args[3], args[4], args[5], ctypes.byref(a)) == 0
        assert L.tt_verify_workspace_size(args[0], args[1], ctypes.byref(v)) == 0
        assert n.value == max(a.value, v.value)
    assert L.tt_step_workspace_size(8, 10, 4096, 4096, -1, 16, ctypes.byref(n)) == tt.TT_EUNSUPPORTED


def test_invalid_arguments_return_before_launch():
    L = tt.lib()
    P = ctypes.c_void_p
    dummy = P(0x1000)  # never dereferenced: every call below fails validation first
    v = tt.c_tt_vocab(0x1000, 0x1000, 10, 8)
    assert L.tt_align(None, ctypes.byref(v), 1, dummy, dummy, dummy, dummy, 4, 4, 8,
                      dummy, dummy, dummy, dummy, None, 0, None) == tt.TT_EINVAL
    assert L.tt_align(ctypes.byref(v), ctypes.byref(v), -1, dummy, dummy, dummy, dummy, 4, 4, 8,
                      dummy, dummy, dummy, dummy, None, 0, None) == tt.TT_EINVAL
    big = tt.c_tt_vocab(0x1000, 0x1000, 10, 65)
    assert L.tt_align(ctypes.byref(big), ctypes.byref(v), 1, dummy, dummy, dummy, dummy, 4, 4, 8,
                      dummy, dummy, dummy, dummy, None, 0, None) == tt.TT_EUNSUPPORTED
    assert L.tt_align(ctypes.byref(v), ctypes.byref(v), 1, None, dummy, dummy, dummy, 4, 4, 8,
                      dummy, dummy, dummy, dummy, None, 0, None) == tt.TT_EINVAL
    assert L.tt_align(ctypes.byref(v), ctypes.byref(v), 0, None, None, None, None, 4, 4, 8,
                      None, None, None, None, None, 0, None) == tt.TT_OK  # empty batch
    assert L.tt_transfer(1, 10, dummy, dummy, dummy, dummy, dummy, 5, dummy, None) == tt.TT_EINVAL
    assert L.tt_transfer(1, 10, dummy, None, dummy, dummy, dummy, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_verify(1, 10, dummy, dummy, dummy, dummy, 9, dummy, dummy, 4, dummy, dummy, None,
                       dummy, 1 << 20, None) == tt.TT_EINVAL  # ld < v_t
    assert L.tt_verify(1, 10, dummy, dummy, dummy, dummy, 10, dummy, dummy, -1, dummy, dummy, None,
                       dummy, 1 << 20, None) == tt.TT_EINVAL
    assert L.tt_verify(1, 10, dummy, dummy, dummy, dummy, 10, dummy, dummy, 4, dummy, dummy, None,
                       dummy, 0, None) == tt.TT_EWORKSPACE
    assert L.tt_verify(1, 10, None, dummy, dummy, dummy, 10, dummy, dummy, 4, dummy, dummy, None,
                       dummy, 1 << 20, None) == tt.TT_EINVAL

    def dense(n=1, v=10, ld_d=10, ld_t=10, max_m=4, ids=dummy, ws=1 << 20):
        return L.tt_verify_dense(n, v, ids, dummy, dummy, ld_d, dummy, ld_t, dummy, dummy, max_m, dummy, dummy,
                                 None, dummy, ws, None)
    assert dense(ld_d=9) == tt.TT_EINVAL
    assert dense(ld_t=9) == tt.TT_EINVAL
    assert dense(v=0) == tt.TT_EINVAL
    assert dense(max_m=-1) == tt.TT_EINVAL
    assert dense(n=-1) == tt.TT_EINVAL
    assert dense(ids=None) == tt.TT_EINVAL
    assert dense(ws=0) == tt.TT_EWORKSPACE
    assert dense(n=0, ids=None) == tt.TT_OK

    assert L.tt_delta_histogram(1, dummy, dummy, dummy, dummy, 0, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_histogram(1, dummy, dummy, dummy, dummy, 8193, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_histogram(1, dummy, None, dummy, dummy, 8, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_histogram(-1, dummy, dummy, dummy, dummy, 8, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_histogram(1, dummy, dummy, dummy, dummy, 8, None, None) == tt.TT_EINVAL

    n = ctypes.c_size_t(0)
    assert L.tt_token_index_size(0, ctypes.byref(n)) == tt.TT_EINVAL
    # 16-byte slots (a power of two >= 4 x the tokens) and a filter of 2 bits per slot
    assert L.tt_token_index_size(1000, ctypes.byref(n)) == 0 and n.value == 16 * 4096 + 4096 // 4
    assert L.tt_token_index_size(151936, ctypes.byref(n)) == 0 and n.value == 16 * (1 << 20) + (1 << 20) // 4
    assert L.tt_token_index_build(ctypes.byref(big), dummy, 1 << 30, None) == tt.TT_EUNSUPPORTED
    assert L.tt_token_index_build(ctypes.byref(v), P(0x1004), 1 << 30, None) == tt.TT_EINVAL  # not 16-byte aligned
    assert L.tt_token_index_build(ctypes.byref(v), dummy, 16, None) == tt.TT_EWORKSPACE
    assert L.tt_retokenize_workspace_size(4, 0, ctypes.byref(n)) == tt.TT_EINVAL
    assert L.tt_retokenize_workspace_size(4, 10, ctypes.byref(n)) == 0 and n.value >= 4 * 4 + 4 * 40

    def retok(n=1, max_bytes=64, max_m=16, index=dummy, ib=1 << 20, ws=1 << 20, ids=dummy, vt=ctypes.byref(v)):
        return L.tt_retokenize(ctypes.byref(v), vt, index, ib, n, ids, dummy, max_bytes, max_m, dummy, dummy, dummy,
                               ws, None)
    assert retok(max_bytes=0) == tt.TT_EINVAL
    assert retok(max_bytes=4097) == tt.TT_EINVAL
    assert retok(max_m=0) == tt.TT_EINVAL
    assert retok(index=P(0x1008)) == tt.TT_EINVAL
    assert retok(ib=16) == tt.TT_EINVAL
    assert retok(ws=4) == tt.TT_EWORKSPACE
    assert retok(ids=None) == tt.TT_EINVAL
    assert retok(n=-1) == tt.TT_EINVAL
    assert retok(vt=ctypes.byref(big)) == tt.TT_EUNSUPPORTED

    def step(vd=ctypes.byref(v), n=1, v_d=10, v_t=10, ld_d=10, ld_t=10, max_m=4, ids=dummy, ws=1 << 30):
        return L.tt_step(vd, ctypes.byref(v), n, v_d, v_t, ids, dummy, dummy, dummy, 4, max_m, 8,
                         dummy, ld_d, dummy, ld_t, dummy, dummy, dummy, dummy, dummy, dummy, dummy,
                         dummy, dummy, None, dummy, ws, None)
    assert step(vd=None) == tt.TT_EINVAL
    assert step(n=-1) == tt.TT_EINVAL
    assert step(ld_d=9) == tt.TT_EINVAL
    assert step(ld_t=9) == tt.TT_EINVAL
    assert step(max_m=0) == tt.TT_EINVAL
    assert step(ids=None) == tt.TT_EINVAL
    assert step(ws=16) == tt.TT_EWORKSPACE
    assert step(vd=ctypes.byref(big)) == tt.TT_EUNSUPPORTED
    assert step(n=0) == tt.TT_OK

    def isect(vd=ctypes.byref(v), ia=dummy, ib_d=1 << 20, it=dummy, ib_t=1 << 20, d2t=dummy, t2d=dummy):
        return L.tt_vocab_intersection(vd, ia, ib_d, ctypes.byref(v), it, ib_t, d2t, t2d, None)
    assert isect(vd=None) == tt.TT_EINVAL
    assert isect(ia=None) == tt.TT_EINVAL
    assert isect(it=P(0x1008)) == tt.TT_EINVAL  # not 16-byte aligned
    assert isect(ib_d=16) == tt.TT_EINVAL
    assert isect(ib_t=16) == tt.TT_EINVAL
    assert isect(t2d=None) == tt.TT_EINVAL
    assert isect(vd=ctypes.byref(big)) == tt.TT_EUNSUPPORTED

    def logits(n=1, v=10, ld=10, max_m=4, it=dummy, lg=dummy):
        return L.tt_verify_logits(n, v, dummy, dummy, dummy, lg, ld, it, None, dummy, dummy, max_m, dummy, dummy,
                                  None)
    assert logits(n=-1) == tt.TT_EINVAL
    assert logits(v=0) == tt.TT_EINVAL
    assert logits(ld=9) == tt.TT_EINVAL
    assert logits(max_m=-1) == tt.TT_EINVAL
    assert logits(it=None) == tt.TT_EINVAL
    assert logits(lg=None) == tt.TT_EINVAL
    assert logits(v=(1 << 23) + 1, ld=(1 << 23) + 1) == tt.TT_EUNSUPPORTED
    assert logits(n=0, lg=None) == tt.TT_OK

    def tli(n=2, v_d=10, v_t=12, ld_d=10, ld_q=12, d2t=dummy, q=dummy):
        return L.tt_tli_proposal(n, v_d, v_t, d2t, dummy, dummy, ld_d, q, ld_q, None)
    assert tli(n=-1) == tt.TT_EINVAL
    assert tli(v_d=0) == tt.TT_EINVAL
    assert tli(v_t=0) == tt.TT_EINVAL
    assert tli(ld_d=9) == tt.TT_EINVAL
    assert tli(ld_q=11) == tt.TT_EINVAL
    assert tli(d2t=None) == tt.TT_EINVAL
    assert tli(q=None) == tt.TT_EINVAL
    assert tli(n=0, q=None) == tt.TT_OK

    def vtli(n=2, v_d=10, v_t=12, ld_d=10, ld_t=12, max_m=4, t2d=dummy, q=dummy, mass=None):
        return L.tt_verify_tli(n, v_d, v_t, dummy, t2d, dummy, dummy, q, ld_d, mass, dummy, ld_t, dummy, dummy,
                               max_m, dummy, dummy, None)
    assert vtli(n=-1) == tt.TT_EINVAL
    assert vtli(v_d=0) == tt.TT_EINVAL
    assert vtli(v_t=0) == tt.TT_EINVAL
    assert vtli(ld_d=9) == tt.TT_EINVAL
    assert vtli(ld_t=11) == tt.TT_EINVAL
    assert vtli(max_m=-1) == tt.TT_EINVAL
    assert vtli(max_m=65537) == tt.TT_EINVAL
    assert vtli(t2d=None) == tt.TT_EINVAL
    assert vtli(q=None) == tt.TT_EINVAL
    assert vtli(v_t=(1 << 21) + 1, ld_t=(1 << 21) + 1) == tt.TT_EUNSUPPORTED
    assert vtli(n=0, q=None) == tt.TT_OK


def test_binding_refuses_host_tensors():
    torch = pytest.importorskip("torch")
    with pytest.raises(ValueError):
        tt._ptr(torch.zeros(3, dtype=torch.int32), torch.int32, "x")


def test_delta_quantile_argument_checks():
    """App. K's quantile call rejects bad sizes and fractions on the host."""
    L = tt.lib()
    dummy = ctypes.c_void_p(16)
    assert L.tt_delta_quantile(None, 8, 9, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8, 9, 10, None, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 0, 9, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8193, 9, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8, 11, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8, -1, 10, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8, 1, 0, dummy, None) == tt.TT_EINVAL
    assert L.tt_delta_quantile(dummy, 8, 1, 65537, dummy, None) == tt.TT_EINVAL


def test_calls_with_an_optional_workspace():
    """tt_verify_logits_ws and tt_verify_tli_ws: size queries, a workspace that is too small, and the checks that
    they share with the calls without one."""
    L = tt.lib()
    P = ctypes.c_void_p
    dummy = P(0x1000)  # never dereferenced: every call below fails validation first, or is empty
    n = ctypes.c_size_t(7)
    lsize = lambda *a: L.tt_verify_logits_workspace_size(*a, ctypes.byref(n))  # noqa: E731
    assert L.tt_verify_logits_workspace_size(4, 40000, 4, 0, None) == tt.TT_EINVAL
    for bad in ((-1, 40000, 4, 0), (4, 0, 4, 0), (4, 40000, -1, 0), (4, 40000, 65537, 0)):
        assert lsize(*bad) == tt.TT_EINVAL, bad
    assert lsize(4, (1 << 23) + 1, 4, 0) == tt.TT_EUNSUPPORTED
    # few streams: per row the estimates, and per stream the selected row's 40 exact chunk sums
    assert lsize(4, 40000, 4, 0) == 0 and n.value >= 4 * 5 * 8 + 4 * 40 * 8
    assert lsize(4, 40000, 4, 1) == 0 and n.value >= 4 * 40 * 8
    for none in ((0, 40000, 4, 0), (4, 40000, 0, 0), (513, 40000, 4, 0), (4, 20000, 4, 1), (129, 40000, 4, 1), (65, 40000, 1, 0)):
        n.value = 7
        assert lsize(*none) == 0 and n.value == 0, none  # the one kernel is the better one
    assert lsize(512, 1 << 23, 65536, 0) == 0 and n.value < 64 << 20

    def logits(ws=dummy, size=1 << 30, n=4, v=40000, ld=40000, max_m=4, it=dummy, lse=None):
        return L.tt_verify_logits_ws(n, v, dummy, dummy, dummy, dummy, ld, it, lse, dummy, dummy, max_m, dummy, dummy, ws,
                                     size, None)
    assert logits(n=-1) == tt.TT_EINVAL
    assert logits(ld=39999) == tt.TT_EINVAL
    assert logits(max_m=65537) == tt.TT_EINVAL
    assert logits(it=None) == tt.TT_EINVAL
    assert logits(v=(1 << 23) + 1, ld=(1 << 23) + 1) == tt.TT_EUNSUPPORTED
    assert logits(n=0, it=None) == tt.TT_OK
    assert logits(n=0, ws=None, size=0) == tt.TT_OK
    for lse in (None, dummy):
        assert lsize(4, 40000, 4, 0 if lse is None else 1) == 0
        assert logits(size=n.value - 1, lse=lse) == tt.TT_EWORKSPACE
        assert logits(size=0, lse=lse) == tt.TT_EWORKSPACE

    tsize = lambda *a: L.tt_verify_tli_workspace_size(*a, ctypes.byref(n))  # noqa: E731
    assert L.tt_verify_tli_workspace_size(4, 40000, None) == tt.TT_EINVAL
    assert tsize(-1, 40000) == tt.TT_EINVAL
    assert tsize(4, 0) == tt.TT_EINVAL
    assert tsize(4, (1 << 21) + 1) == tt.TT_EUNSUPPORTED
    for none in ((0, 40000), (4, 31744), (65, 40000), (129, 151936)):
        n.value = 7
        assert tsize(*none) == 0 and n.value == 0, none
    assert tsize(128, 151936) == 0 and n.value >= 128 * (8 + 149 * 8)

    def tli(ws=dummy, size=1 << 30, n=4, v_d=10, v_t=40000, ld_d=10, ld_t=40000, max_m=4, q=dummy, mass=None):
        return L.tt_verify_tli_ws(n, v_d, v_t, dummy, dummy, dummy, dummy, q, ld_d, mass, dummy, ld_t, dummy, dummy, max_m,
                                  dummy, dummy, ws, size, None)
    assert tli(n=-1) == tt.TT_EINVAL
    assert tli(ld_t=39999) == tt.TT_EINVAL
    assert tli(q=None) == tt.TT_EINVAL
    assert tli(v_t=(1 << 21) + 1, ld_t=(1 << 21) + 1) == tt.TT_EUNSUPPORTED
    assert tli(n=0, ws=None, size=0) == tt.TT_OK
    assert tsize(4, 40000) == 0
    assert tli(size=n.value - 1) == tt.TT_EWORKSPACE
    assert tli(size=n.value - 1, mass=dummy) == tt.TT_EWORKSPACE


def test_package_imports_without_torch():
    """The workload generator and the build script need no torch."""
    code = ("import sys; sys.modules['torch'] = None\n"
            "import paper_2510_15545_amd as tt\n"
            "from paper_2510_15545_amd import build, synth\n"
            "assert tt.lib().tt_version() >= 100 and synth.make(1, n_streams=1).n == 1 and build.sources()")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


def test_stream_handles(monkeypatch):
    """The caller's stream, the current stream's raw handle, and the current stream where torch has no such call."""
    raw = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda device: 100 + device)
    cuda = types.SimpleNamespace(current_device=lambda: 2, current_stream=lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(tt, "torch", types.SimpleNamespace(_C=raw, cuda=cuda))
    assert tt._stream_handle(types.SimpleNamespace(cuda_stream=5)) == 5
    assert tt._stream_handle(None) == 102
    monkeypatch.setattr(tt, "torch", types.SimpleNamespace(_C=types.SimpleNamespace(), cuda=cuda))
    assert tt._stream_handle(None) == 77
