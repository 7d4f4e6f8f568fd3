"""Kernels at the sizes where their tiles, waves and dispatch rules change,
against the oracle in float64, through the C ABI.

fp32 results are judged by the norm of the error over the norm of the result.
A running sum of n independent terms errs by about sqrt(n / 6) 2^-24 in the norm
when each rounding is uniform over half an ulp of a partial sum that grows as a
square root: 2.0e-7 for the 64 products of a READ leaf (32 rows of dW and W0), 7.8e-7
for the longest chain here, the 1024 evidence rows of an fp32 WRITE (one accumulator
over the whole chunk; 1.5e-7 for 40 rows).  The adapter kernels' chains have at most
16 products, and trees and short second stages add less, so 1e-6 holds for all.
bf16 results add one rounding, 2^-9 at most per value (1.7e-3 in the norm; 4e-3
bound).
"""

import dataclasses

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


# One tile of evidence rows a block for an owner alone; two and four, past one
# round of blocks, for the group
@pytest.mark.parametrize("d_ff,d_model,io,state,rank,chunk", [
    (1032, 2056, "bf16", "f32", 16, 100), (1032, 2056, "f32", "f32", 5, 145), (1032, 2056, "bf16", "bf16", 17, 100)])
def test_adapter_write_alone_has_the_groups_bits(d_ff, d_model, io, state, rank, chunk):
    wl = small_workload(d_ff, d_model, io, state, 9)
    say("adapter write alone and in a group", d_ff, d_model, io, state, rank, chunk)
    sess = Session(wl, TensorSource(wl), backend=ADA, rank=rank)
    group = list(range(9))[::-1]
    dev = {r: [to_device(t, io) for t in evidence(wl, chunk, r)] for r in group}
    assert write_group(sess, group, 0, chunk, [dev[r][0] for r in group], [dev[r][1] for r in group]) == R.RWTTT_OK
    assert R.rwttt_rollback(sess.ctx, group) == R.RWTTT_OK
    torch.cuda.synchronize()
    want = {r: sess.shadow(r, 0).clone() for r in group}
    for r in group:
        sess.shadow(r, 0).zero_()
        assert write_group(sess, [r], 0, chunk, [dev[r][0]], [dev[r][1]]) == R.RWTTT_OK
        assert R.rwttt_rollback(sess.ctx, [r]) == R.RWTTT_OK
        torch.cuda.synchronize()
        assert torch.equal(sess.shadow(r, 0), want[r]), r


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


# fp32 evidence: the smallest matrix, one block of 256 x 64 and one row or
# column group past it, ragged waves; chunk: one, around a matrix step of 4 and
# a group of 16, a long one; rows: the last with 64, the first with 128 and with
# 256 rows per partial of the token
F32_WRITES = [
    (4096, 264, "f32", 2), (4104, 136, "f32", 3), (8200, 72, "f32", 6),
    (8, 8, "f32", 1), (256, 64, "f32", 4), (264, 72, "bf16", 5), (248, 56, "f32", 15), (512, 136, "bf16", 16),
    (776, 200, "f32", 17), (1032, 1032, "f32", 130), (264, 72, "f32", 1024),
]


@pytest.mark.parametrize("token", [True, False])
@pytest.mark.parametrize("d_ff,d_model,state,chunk", F32_WRITES)
def test_f32_write_edges(d_ff, d_model, state, chunk, token):
    wl = small_workload(d_ff, d_model, "f32", state, 3)
    say("f32 write edge", d_ff, d_model, state, chunk, token)
    src = TensorSource(wl)
    sess = Session(wl, src, tail_rows=0)
    group = [2, 0]
    ev = [evidence(wl, chunk, r) for r in group]
    X = draw((3, d_ff), 1.0, "f32", wl.seed, (63, chunk))
    xd = to_device(X, "f32")
    y = torch.full((3, d_model), 7.0, device="cuda")
    st = write_group(sess, group, 0, chunk, [to_device(z, "f32") for z, _ in ev],
                     [to_device(g, "f32") for _, g in ev], None, *((xd, y) if token else ()))
    assert st == R.RWTTT_OK
    torch.cuda.synchronize()
    W0 = O.widen(src.w0(0), "f32")
    for r, (Z, G) in zip(group, ev):
        D = O.widen(src.dw_init(r, 0), state)
        want = O.write_candidate(D, O.widen(Z, "f32"), O.widen(G, "f32"), wl.eta)
        assert rel_norm(host_f64(sess.shadow(r, 0), state), want) <= norm_tol(state), r
        if token:
            assert rel_norm(host_f64(y[r], "f32"), O.read_apply(O.widen(X[r], "f32"), W0, D)) <= 1e-6, r
    assert torch.all(y[1] == 7.0) and (token or torch.all(y == 7.0))


def test_f32_write_keeps_non_finite_evidence_in_its_place():
    wl = small_workload(264, 72, "f32", "f32", 1)
    sess = Session(wl, TensorSource(wl), tail_rows=0)
    Z, G = evidence(wl, 5, 0)
    zd, gd = to_device(Z, "f32"), to_device(G, "f32")
    zd[4, 263], gd[4, 71] = float("inf"), float("nan")
    assert write_group(sess, [0], 0, 5, [zd], [gd]) == R.RWTTT_OK
    bad = ~torch.isfinite(sess.shadow(0, 0))
    want = torch.zeros_like(bad)
    want[263, :] = want[:, 71] = True
    assert torch.equal(bad, want)


# READs of up to 1536 rows run as one launch for 38 MB of state and W0 and 1024
# blocks, as two above: a group on each side must give an owner the same bits.
# Rows: one leaf of 8, one leaf per row group (1024) and past it, the limit and past
# it (always two launches); the last column tile is ragged
READ_ROUTES = [
    (264, 4104, "bf16", "f32", 12), (1024, 2056, "bf16", "bf16", 9), (1032, 2056, "bf16", "f32", 5),
    (1536, 1032, "f32", "f32", 8), (1544, 1032, "bf16", "f32", 8), (3600, 520, "f32", "bf16", 3),
    (3600, 1512, "f32", "bf16", 7),                          # four waves in a group, eight alone
    (8, 8, "f32", "f32", 2), (16, 72, "bf16", "f32", 3), (8, 8200, "bf16", "bf16", 8), (16, 8200, "bf16", "f32", 6),
]


@pytest.mark.parametrize("d_ff,d_model,io,state,n", READ_ROUTES)
def test_read_routes_agree_bit_for_bit(d_ff, d_model, io, state, n):
    wl = small_workload(d_ff, d_model, io, state, n)
    say("read route", d_ff, d_model, io, state, n)
    src = TensorSource(wl)
    sess = Session(wl, src, tail_rows=2)
    X = draw((n, d_ff), 1.0, io, wl.seed, (64, n))
    xd = to_device(X, io)
    group = list(range(n))[::-1]
    y = [torch.full((n, d_model), 7.0, device="cuda", dtype=xd.dtype) for _ in range(2)]
    read_group(sess, group, 0, xd, y[0])
    for r in range(n):                                       # alone, with the tail append
        st = R.rwttt_read_append(sess.ctx, R.make_group(R.RWTTT_READ, 0, 1), R.u32_array([r]), 0, xd.data_ptr(),
                                 y[1].data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert st == R.RWTTT_OK
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1])
    for r in range(n):
        assert torch.equal(sess.tails[r][0][0], xd[r]) and not sess.tails[r][0][1].any()
    W0 = O.widen(src.w0(0), io)
    for r in (0, n - 1):
        want = O.read_apply(O.widen(X[r], io), W0, O.widen(src.dw_init(r, 0), state))
        assert rel_norm(host_f64(y[0][r], io), want) <= norm_tol(io), r


# bf16 evidence without a token.  fp32 state, register operands: the smallest
# matrix, a tile of 64 x 64 and its remainders (8 rows in a lane's second run,
# one column group past the tile), a count of tiles no block of four divides;
# chunk: one, a group of 16 and past it, the last of this path and the first three
# counts of GEMM stages past it (13 to 15: the last stage in each of its three buffers).  bf16 state: streaming and GEMM on both sides of the small-state line
# (2.2 M elements of a group, one item a block), chunks of one and two GEMM stages
# of 32 ranks; a row of GEMM tiles and a column of them, fewer than the XCDs
ROWS_WRITES = [
    (8, 8, "f32", 1), (64, 64, "f32", 16), (72, 72, "f32", 17), (136, 328, "f32", 33), (248, 1032, "f32", 64),
    (520, 264, "f32", 384), (520, 264, "f32", 385), (264, 136, "f32", 417), (264, 264, "f32", 449), (8, 8, "bf16", 1), (264, 136, "bf16", 31), (520, 136, "bf16", 33),
    (264, 264, "bf16", 64), (2048, 512, "bf16", 17), (2056, 512, "bf16", 64), (1544, 1032, "bf16", 33),
    (72, 16392, "bf16", 64), (8200, 72, "bf16", 20), (264, 4104, "bf16", 70),
]


@pytest.mark.parametrize("d_ff,d_model,state,chunk", ROWS_WRITES)
def test_bf16_write_without_token_edges(d_ff, d_model, state, chunk):
    wl = small_workload(d_ff, d_model, "bf16", state, 3)
    say("bf16 write edge", d_ff, d_model, state, chunk)
    src = TensorSource(wl)
    sess = Session(wl, src)
    group = [2, 0]
    ev = [evidence(wl, chunk, r) for r in group]
    guard = sess.slots[1][0][1].fill_(7.0)                   # an owner outside the group
    st = write_group(sess, group, 0, chunk, [to_device(z, "bf16") for z, _ in ev],
                     [to_device(g, "bf16") for _, g in ev])
    assert st == R.RWTTT_OK
    torch.cuda.synchronize()
    for r, (Z, G) in zip(group, ev):
        D = O.widen(src.dw_init(r, 0), state)
        want = O.write_candidate(D, O.widen(Z, "bf16"), O.widen(G, "bf16"), wl.eta)
        assert rel_norm(host_f64(sess.shadow(r, 0), state), want) <= norm_tol(state), r
    assert torch.all(guard == 7.0)


def test_bf16_write_keeps_non_finite_evidence_in_its_place():
    wl = small_workload(136, 72, "bf16", "f32", 1)
    sess = Session(wl, TensorSource(wl))
    Z, G = evidence(wl, 21, 0)
    zd, gd = to_device(Z, "bf16"), to_device(G, "bf16")
    zd[20, 135], gd[20, 71] = float("inf"), float("nan")
    assert write_group(sess, [0], 0, 21, [zd], [gd]) == R.RWTTT_OK
    bad = ~torch.isfinite(sess.shadow(0, 0))
    want = torch.zeros_like(bad)
    want[135, :] = want[:, 71] = True
    assert torch.equal(bad, want)


# the routes of a bf16 WRITE with a fused token and fp32 state: register operands
# from 512 columns, up to 4096 rows and 4 M elements, streaming outside
TOKEN_WRITES = [
    (8, 512, 1), (72, 520, 16), (264, 776, 17), (1032, 520, 64), (4096, 512, 33), (4096, 1024, 31),
    (8, 8, 1), (264, 504, 17), (4104, 512, 33), (4096, 1032, 31),
]


@pytest.mark.parametrize("d_ff,d_model,chunk", TOKEN_WRITES)
def test_bf16_write_with_token_edges(d_ff, d_model, chunk):
    """Token and candidate of two owners (slots in reverse owner order) against
    64 bits, and the bits of an owner alone."""
    say("token write", d_ff, d_model, chunk)
    wl = small_workload(d_ff, d_model, "bf16", "f32", 3, eta=0.01)
    src = TensorSource(wl)
    sess = Session(wl, src)
    x = draw((3, d_ff), 1.0, "bf16", wl.seed, (61,))
    xd = to_device(x, "bf16")
    group = [2, 0]
    zs, gs = zip(*(evidence(wl, chunk, r) for r in group))
    zd, gd = [to_device(z, "bf16") for z in zs], [to_device(g, "bf16") for g in gs]
    y = torch.full((3, d_model), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert write_group(sess, group, 0, chunk, zd, gd, x_dev=xd, y_dev=y) == R.RWTTT_OK
    assert R.rwttt_rollback(sess.ctx, group) == R.RWTTT_OK
    torch.cuda.synchronize()
    both = [sess.shadow(r, 0).clone() for r in group]
    w0 = O.widen(src.w0(0), "bf16")
    for i, r in enumerate(group):
        live = O.widen(src.dw_init(r, 0), "f32")
        assert rel_norm(host_f64(y[r], "bf16"), O.read_apply(O.widen(x[r], "bf16"), w0, live)) <= norm_tol("bf16"), r
        want = O.write_candidate(live, O.widen(zs[i], "bf16"), O.widen(gs[i], "bf16"), wl.eta)
        assert rel_norm(host_f64(both[i], "f32"), want) <= norm_tol("f32"), r
        alone = torch.zeros_like(y)
        assert write_group(sess, [r], 0, chunk, [zd[i]], [gd[i]], x_dev=xd, y_dev=alone) == R.RWTTT_OK
        assert R.rwttt_rollback(sess.ctx, [r]) == R.RWTTT_OK
        torch.cuda.synchronize()
        assert torch.equal(alone[r], y[r]) and torch.equal(sess.shadow(r, 0), both[i])
    assert torch.isnan(y[1]).all()


# Every kernel that loads the live state with and without the non-temporal hint:
# a context of few owners, and one whose states do not fit the 256 MB cache.  An
# owner must also have the same bits alone and in a group, on both sides of the
# rules that look at the group.
BOTH_HINTS = [
    # d_ff, d_model, io, state, chunk (0: READ), token, group, owners of the large context
    (2056, 1032, "bf16", "f32", 0, False, 2, 32),     # READ: eight waves, four alone
    (2056, 1032, "bf16", "bf16", 0, False, 3, 64),
    (1024, 2056, "bf16", "f32", 0, False, 5, 32),     # two launches, one alone
    (2056, 1032, "f32", "bf16", 0, False, 3, 64),
    (2000, 776, "bf16", "f32", 33, True, 3, 44),      # register operands with token
    (4104, 512, "bf16", "f32", 64, True, 3, 32),      # streaming with token
    (2056, 1032, "bf16", "bf16", 17, True, 3, 64),
    (2000, 776, "bf16", "f32", 100, False, 3, 44),    # register operands
    (520, 264, "bf16", "f32", 400, True, 2, 500),     # READ, then the GEMM with fp32 state
    (2000, 2000, "bf16", "f32", 345, False, 8, 20),   # GEMM, register operands alone
    (2048, 1016, "bf16", "f32", 300, True, 8, 40),    # ... after a READ
    (1544, 1032, "bf16", "bf16", 33, False, 3, 84),   # GEMM, streaming alone
    (64, 16392, "bf16", "bf16", 33, False, 8, 130),   # ... few rows
    (4096, 264, "f32", "f32", 5, True, 3, 64),        # fp32 evidence: blocks of 64 rows
    (4104, 520, "f32", "f32", 40, True, 3, 32),       # ... of 128
    (8200, 264, "f32", "bf16", 17, True, 3, 64),      # ... of 256
    (4104, 520, "f32", "f32", 40, False, 3, 32),
]


@pytest.mark.parametrize("d_ff,d_model,io,state,chunk,token,n,many", BOTH_HINTS)
def test_same_bits_with_either_cache_hint_and_in_any_group(d_ff, d_model, io, state, chunk, token, n, many):
    say("cache hint", d_ff, d_model, io, state, chunk, token)
    wl = small_workload(d_ff, d_model, io, state, n)
    src = TensorSource(wl)
    small = Session(wl, src)
    large = Session(dataclasses.replace(wl, n_owners=many), None, max_group=n)
    large.w0[0].copy_(small.w0[0])
    for r in range(n):
        large.slots[r][0][0].copy_(small.slots[r][0][0])
    x = draw((many, d_ff), 1.0, io, wl.seed, (65, chunk))
    xd = to_device(x, io)
    ev = [evidence(wl, chunk, r) for r in range(n)] if chunk else []
    dev = [(to_device(z, io), to_device(g, io)) for z, g in ev]

    def call(sess, owners):
        """{owner: (token or y, candidate)}"""
        y = torch.full((many, d_model), 7.0, device="cuda", dtype=xd.dtype)
        if not chunk:
            read_group(sess, owners, 0, xd, y)
        else:
            assert write_group(sess, owners, 0, chunk, [dev[r][0] for r in owners], [dev[r][1] for r in owners], None,
                               *((xd, y) if token else ())) == R.RWTTT_OK
            assert R.rwttt_rollback(sess.ctx, owners) == R.RWTTT_OK
        torch.cuda.synchronize()
        assert torch.all(y[n:] == 7.0)
        return {r: (y[r].clone(), sess.shadow(r, 0).clone() if chunk else y[r]) for r in owners}

    group = list(range(n))[::-1]
    want = call(small, group)
    runs = [call(large, group)] + [call(sess, [r]) for sess in (small, large) for r in group]
    for run in runs:
        for r, (y, cand) in run.items():
            assert torch.equal(y, want[r][0]) and torch.equal(cand, want[r][1]), r
    live = O.widen(src.dw_init(0, 0), state)
    if token or not chunk:
        ref = O.read_apply(O.widen(x[0], io), O.widen(src.w0(0), io), live)
        assert rel_norm(host_f64(want[0][0], io), ref) <= norm_tol(io)
    if chunk:
        ref = O.write_candidate(live, O.widen(ev[0][0], io), O.widen(ev[0][1], io), wl.eta)
        assert rel_norm(host_f64(want[0][1], state), ref) <= norm_tol(state)


# One WRITE path each: register operands with a token and without, streaming, fp32
# evidence with 64 and 256 rows per token partial, READ then the GEMM
TWO_STREAMS = [
    (2000, 776, "bf16", "f32", 33, True), (2000, 776, "bf16", "f32", 100, False), (4104, 512, "bf16", "f32", 64, True),
    (4096, 264, "f32", "f32", 5, True), (8200, 264, "f32", "f32", 17, True), (1000, 264, "bf16", "bf16", 70, True),
]


@pytest.mark.parametrize("d_ff,d_model,io,state,chunk,token", TWO_STREAMS)
def test_writes_and_reads_of_disjoint_owners_on_two_streams(d_ff, d_model, io, state, chunk, token):
    """Two WRITEs, then a WRITE beside a READ, overlapping on two streams with
    disjoint owners: the bits of the same calls one after the other."""
    say("two streams", d_ff, d_model, io, state, chunk, token)
    wl = small_workload(d_ff, d_model, io, state, 5)
    src = TensorSource(wl)
    sess = Session(wl, src)
    xd = to_device(draw((5, d_ff), 1.0, io, wl.seed, (66,)), io)
    dev = {r: [to_device(t, io) for t in evidence(wl, chunk, r)] for r in range(5)}
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def write(owners, y):
        assert write_group(sess, owners, 0, chunk, [dev[r][0] for r in owners], [dev[r][1] for r in owners], None,
                           *((xd, y) if token else ())) == R.RWTTT_OK

    def read(owners, y):
        read_group(sess, owners, 0, xd, y)

    for first, second in ((write, write), (write, read)):
        results = []
        for overlap in (False, True, True, True):
            y = [torch.zeros((5, d_model), device="cuda", dtype=xd.dtype) for _ in range(2)]
            for r in range(5):
                sess.shadow(r, 0).zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(streams[0]):
                first([3, 0], y[0])
            if not overlap:
                torch.cuda.synchronize()
            with torch.cuda.stream(streams[1]):
                second([1, 4, 2], y[1])
            torch.cuda.synchronize()
            assert R.rwttt_rollback(sess.ctx, [3, 0] + ([1, 4, 2] if second is write else [])) == R.RWTTT_OK
            results.append(y + [sess.shadow(r, 0).clone() for r in range(5)])
        for got in results[1:]:
            assert all(torch.equal(a, b) for a, b in zip(got, results[0]))
