"""The acceptance probability of the bf16-logits verification in numpy, for tests that set q beside it."""
import numpy as np


def accept_probs(V, case):
    """P of every proposal (to within an fp32 step or two) and its row: the specified arithmetic in numpy."""
    ids, off, q, bits, it, ua, us, Ms = case
    f32, stream = np.float32, np.repeat(np.arange(len(Ms)), Ms)
    rows = np.arange(len(ids)) + stream
    coef = [float.fromhex(h) for h in ("0x1.5d87fep-10", "0x1.3b2ab6p-7", "0x1.c6b08ep-5", "0x1.ebfbe0p-3", "0x1.62e430p-1")] + [1.0]
    P = np.zeros(len(ids))
    for k, r in enumerate(rows):
        x = (bits[r, :V].astype(np.uint32) << 16).view(f32).astype(np.float64)
        c = float(f32(it[stream[k]] * f32(1.4426950408889634)))
        b31 = float(f32(31.0) - (x * c).astype(f32).max())
        z = np.clip((x * c + b31).astype(f32), -1, 31).astype(np.float64)
        kz = np.rint(z)
        p = np.full(len(z), coef[0])
        for h in coef[1:]:
            p = (p * (z - kz) + h).astype(f32).astype(np.float64)
        w = p * 2.0 ** kz
        t = ids[k]
        P[k] = (w[t] if x[t] * c + b31 >= 0 else 0.0) / np.floor(w).sum()
    return P
