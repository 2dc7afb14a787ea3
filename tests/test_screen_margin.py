"""The error bound of the screen's estimate of P (csrc/logits.hip: kMargin's derivation), on a model of its
arithmetic in which every hardware exponential is one unit too large, then one too small."""
import numpy as np
import pytest

from test_oracle_logits import bf16_bits
from util_logits import accept_probs

F32 = np.float32
BOUND = 1.1e-4  # kMargin is 2e-4


def estimate(x, c, t, unit):
    """e / s of one row as the screen forms it: a lane's 16 logits of every chunk, its sum rescaled where its largest y
    rises; then the lanes, pairwise.  One wave takes all chunks, the most that a lane can have."""
    exp2 = lambda v: np.nextafter(np.exp2(v.astype(np.float64)).astype(F32), F32(unit) * F32(np.inf)).astype(F32)  # noqa: E731
    fma = lambda v, m: (v.astype(np.float64) * float(c) - m).astype(F32)  # noqa: E731
    nc = -(-len(x) // 1024)
    chunks = np.full(nc * 1024, -np.inf, F32)
    chunks[:len(x)] = x
    m, s = np.full(64, -3e38, F32), np.zeros(64, F32)
    for k in chunks.reshape(nc, 64, 16):
        mn = np.maximum(m, (k.max(1) * F32(c)).astype(F32))
        term = np.zeros(64, F32)
        for j in range(16):
            term = (term + exp2(fma(k[:, j], mn.astype(np.float64)))).astype(F32)
        s = ((s * exp2(m - mn)).astype(F32) + term).astype(F32)
        m = mn
    M = m.max()
    s = (s * exp2(m - M)).astype(F32)
    while len(s) > 1:
        s = (s[: len(s) // 2] + s[len(s) // 2:]).astype(F32)
    return float(exp2(fma(x[t:t + 1], float(M)))[0]) / float(s[0])


@pytest.mark.parametrize("level", [-350.0, 0.0, 300.0])
@pytest.mark.parametrize("unit", [-1, 1])
def test_estimate_stays_within_the_stated_bound(level, unit):
    """256 chunks of a lane, the largest logit a bf16 step higher in each (as far as bf16 has steps there)."""
    V = 256 * 1024
    x = np.repeat(np.linspace(level, level + 20.0, 256, dtype=F32), 1024)
    bits = bf16_bits(x[None])
    x = (bits[0].astype(np.uint32) << 16).view(F32)
    it = np.float32([1.0])
    ids = np.int32([V - 1])
    case = (ids, np.int32([0, 1]), None, np.concatenate([bits, bits]), it, None, None, np.array([1]))
    P = accept_probs(V, case)[0]
    err = abs(estimate(x, F32(it[0] * F32(1.4426950408889634)), V - 1, unit) / P - 1.0)
    assert err < BOUND, err
