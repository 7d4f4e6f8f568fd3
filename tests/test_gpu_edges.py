"""Kernels at the sizes where their tiles, waves and dispatch rules change,
against the oracle in float64, through the C ABI.

fp32 results are judged by the norm of the error over the norm of the result:
every fp32 kernel adds each product in a chain of at most 32 roundings of a
running sum plus trees, and such sums of independent terms err by about
sqrt(32) 2^-25 = 1.7e-7 in the norm per stage, so 1e-6 leaves a factor of
three over two stages.  bf16 results add one rounding, 2^-9 at most per value
(1.7e-3 in the norm; 4e-3 bound).
"""

import numpy as np
import pytest
import torch

import oracle as O
from rwttt_inputs import TensorSource, draw
from tests.gpu_util import R, Session, host_f64, read_group, say, small_workload, to_device, write_group

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

ADA = R.RWTTT_DELTA_ADAPTER


def norm_tol(dtype):
    return 1e-6 if dtype == "f32" else 4e-3


def rel_norm(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def evidence(wl, chunk, key):
    Z = draw((chunk, wl.d_ff), 1.0, wl.io_dtype, wl.seed, (61, key))
    G = draw((chunk, wl.d_model), 1.0, wl.io_dtype, wl.seed, (62, key))
    return Z, G


# chunk: below, at and above one group of 16 rows, the four-wave and the
# 128-row limits, the largest; rank: one, both sides of the 16-column tile, odd
# and even above it, the largest; extents: the smallest (8), one slice of 1024
# and one row tile of 64 and just past each
ADAPTER_WRITES = [
    (8, 8, "bf16", "f32", 1, 1), (64, 72, "f32", "f32", 15, 3), (1024, 64, "bf16", "f32", 16, 16),
    (1032, 2056, "bf16", "bf16", 17, 17), (136, 1024, "f32", "f32", 32, 64), (2064, 136, "bf16", "f32", 31, 65),
    (264, 520, "bf16", "f32", 18, 128), (520, 264, "f32", "bf16", 8, 129), (72, 128, "bf16", "f32", 16, 1024),
]


@pytest.mark.parametrize("d_ff,d_model,io,state,rank,chunk", ADAPTER_WRITES)
def test_adapter_write_edges(d_ff, d_model, io, state, rank, chunk):
    wl = small_workload(d_ff, d_model, io, state, 2)
    say("adapter write edge", d_ff, d_model, io, state, rank, chunk)
    src = TensorSource(wl)
    sess = Session(wl, src, backend=ADA, rank=rank)
    group = [1, 0]
    ev = [evidence(wl, chunk, r) for r in group]
    st = write_group(sess, group, 0, chunk, [to_device(z, io) for z, _ in ev], [to_device(g, io) for _, g in ev])
    assert st == R.RWTTT_OK
    torch.cuda.synchronize()
    for r, (Z, G) in zip(group, ev):
        A, B = (O.widen(f, state) for f in src.adapter_init(r, 0, rank))
        got = [host_f64(f, state) for f in sess.factors(sess.shadow(r, 0))]
        for g, want in zip(got, O.adapter_write(A, B, O.widen(Z, io), O.widen(G, io), wl.eta)):
            assert rel_norm(g, want) <= norm_tol(state), r


def test_adapter_write_keeps_non_finite_evidence_in_its_place():
    """An infinite evidence value reaches what it enters and nothing else (rows
    past the chunk and columns past the rank are clamped copies of real ones)."""
    wl = small_workload(72, 136, "bf16", "f32", 1)
    sess = Session(wl, TensorSource(wl), backend=ADA, rank=5)
    Z, G = evidence(wl, 19, 0)
    zd, gd = to_device(Z, "bf16"), to_device(G, "bf16")
    gd[18, 135] = float("inf")
    assert write_group(sess, [0], 0, 19, [zd], [gd]) == R.RWTTT_OK
    a, b = sess.factors(sess.shadow(0, 0))
    assert not torch.isfinite(a).any()                      # P[18] is infinite and enters every row
    assert not torch.isfinite(b[:, 135]).any()
    assert torch.isfinite(b[:, :135]).all()
    assert write_group(sess, [0], 0, 19, [zd], [gd]) == R.RWTTT_E_DIRTY
