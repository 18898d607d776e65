"""Shared helpers of the GPU parity tests: weights on both sides, error norms."""
import numpy as np
import torch

import rollout_inputs as ri
from oracle import oracle as orc

DIM_KEYS = ("hidden", "n_q", "n_kv", "head_dim", "ffn", "qk_norm", "rms_eps", "rope_base")


def dims_of(shape):
    return {k: shape[k] for k in DIM_KEYS}


def storage_dtype(shape):
    return torch.bfloat16 if shape["dtype"] == "bf16" else torch.float32


def make_both(shape, seed, std=0.02):
    """(weights on the storage grid as CPU torch tensors, the same as fp32 numpy for the oracle)."""
    dt = storage_dtype(shape)
    w = ri.make_weights(shape, seed, device="cpu", dtype=dt, std=std)

    def np32(t):
        return np.ascontiguousarray(t.float().numpy())
    wn = {k: (np32(v) if k != "layers" else [{a: np32(b) for a, b in l.items()} for l in v]) for k, v in w.items()}
    return w, wn


def to_device(w, device="cuda:0"):
    return {k: (v.to(device) if k != "layers" else [{a: b.to(device) for a, b in l.items()} for l in v])
            for k, v in w.items()}


def rel_inf(got, ref):
    """max |got - ref| / max |ref| over the last axis (per row)."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    return np.abs(got - ref).max(-1) / np.abs(ref).max(-1)


class ArgmaxCount:
    """Argmax agreement between GPU and oracle logit rows.

    The target asks for logits within a tolerance `tol` (max |diff| / max |ref| per row) AND >= 99 % equal argmaxes.
    Two rows that satisfy the first may still disagree on the argmax when the reference's own top-2 margin lies inside
    the tolerance band, so the count runs over the rows whose reference margin exceeds tol * max |ref| ("decided"
    rows); the figure over all rows is kept for the record.  A disagreement on any row must be between candidates
    whose reference logits differ by at most twice the band (else the logit bound itself is violated).
    """

    def __init__(self, tol):
        self.tol = tol
        self.rows = self.agree = self.decided = self.decided_agree = 0

    def add(self, got, ref):
        got = np.asarray(got, np.float64)
        ref = np.asarray(ref, np.float64)
        a_got, a_ref = int(np.argmax(got)), int(np.argmax(ref))
        band = self.tol * np.abs(ref).max()
        top2 = np.partition(ref, -2)[-2:]
        margin = float(top2[1] - top2[0])
        self.rows += 1
        self.agree += int(a_got == a_ref)
        if margin > band:
            self.decided += 1
            self.decided_agree += int(a_got == a_ref)
        assert ref[a_ref] - ref[a_got] <= 2 * band, (a_got, a_ref, ref[a_ref] - ref[a_got], band)

    def check(self, min_rows=1):
        assert self.decided >= min_rows, (self.decided, self.rows)
        assert self.decided_agree >= 0.99 * self.decided, self.summary()

    def summary(self):
        return (f"argmax agreement {self.decided_agree}/{self.decided} on rows with a margin above the logit tolerance, "
                f"{self.agree}/{self.rows} on all rows")


# Truncated sampling (mirrored from csrc/cut_plan.h; a CPU test compares them): slices per row, and units of 256 logits per slice.
CUT_UNITS_KEPT = 1056
CUT_UNITS_READ_ALL = 32  # units of a slice up to which it is read without a look at their largest logits
CUT_SHAPES = [(252, 3), (8204, 2), (66052, 1), (66052, 3), (300, 9), (300000, 64),                  # (vocabulary, rows): read whole
              (262404, 2), (66052, 64), (151936, 30), (151936, 128), (262144, 96)]                   # unit by unit


def cut_slices(n, vocab):
    return max(1, min((768 if n * vocab >= 9000000 else 512) // n, 32, (vocab + 2047) // 2048))


def cut_groups(n, vocab):  # of four logits, per slice
    return -(-(vocab // 4) // cut_slices(n, vocab))


def cut_units(n, vocab):
    return -(-cut_groups(n, vocab) // 64)


def cut_by_units(n, vocab):
    """Whether the third pass of such a call looks at the units' largest logits."""
    u = cut_units(n, vocab)
    return u > CUT_UNITS_READ_ALL and cut_slices(n, vocab) * u <= CUT_UNITS_KEPT


# Layers and numbers of rows at which a projection's last weight tile is partial: the shape, rows, projection, its tile (row blocks, waves)
# and the row blocks left for the last one.  The planner is asked about them on the CPU, the kernel runs them on the GPU.
PARTIAL_TILES = [
    (dict(hidden=1024, n_q=8, n_kv=2, ffn=1024), 260, "gate_up", (3, 4), 1),
    (dict(hidden=1024, n_q=8, n_kv=2, ffn=1280), 260, "gate_up", (3, 4), 2),
    (dict(hidden=1024, n_q=8, n_kv=2, ffn=2560), 780, "gate_up", (3, 8), 1),
    (dict(hidden=1024, n_q=8, n_kv=2, ffn=3584), 520, "gate_up", (3, 8), 2),
    (dict(hidden=4096, n_q=24, n_kv=8, ffn=768), 385, "qkv", (3, 4), 1),
    (dict(hidden=4096, n_q=16, n_kv=8, ffn=768), 520, "qkv", (3, 4), 2),
    (dict(hidden=4096, n_q=24, n_kv=8, ffn=768), 780, "qkv", (3, 8), 1),
    (dict(hidden=4096, n_q=40, n_kv=8, ffn=768), 520, "qkv", (3, 8), 2),
    (dict(hidden=4096, n_q=32, n_kv=4, ffn=768), 520, "o", (3, 4), 2),
    (dict(hidden=3584, n_q=8, n_kv=2, ffn=8192), 520, "down", (3, 4), 1),
]
# The same for the output projection of a model with hidden 1024: vocabulary, rows, tile; two of four row blocks are left.
PARTIAL_HEAD_TILES = [(24640, 100, (4, 4)), (24640, 200, (4, 8)), (24640, 300, (4, 4)), (12352, 200, (4, 4)), (4160, 300, (4, 4))]
