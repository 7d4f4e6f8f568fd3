"""Which kernel a call takes: the host rules of the library, on the CPU.

A small program over the library's own header answers one query per line.
"""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BIG = 10 ** 9                          # a context that no cache holds
READ_CHUNK, TOKEN_ROWS = 256, 64       # K rows of a READ partial; an owner's token partials at most
DTYPES = [("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32"), ("f32", "bf16")]
# the smallest matrix, ragged and power-of-two ones, the full shapes
SHAPES = [(8, 8), (256, 64), (1000, 264), (256, 4096), (128, 14336), (1024, 1024), (1536, 1032), (1544, 1032),
          (5000, 128), (4104, 1032), (5000, 1528), (8200, 520), (9728, 2560), (14336, 4096)]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "routes_check")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2605_28053_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "routes_check.cpp"), "-o", exe], check=True)

    def query(*lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        answers = out.stdout.splitlines()
        assert len(answers) == len(lines)
        return [a.split() for a in answers]
    return query


def test_an_owners_order_of_addition_does_not_depend_on_the_group(ask):
    """READ: the leaves' size.  A bf16 token of C <= 64: the kernel."""
    for io, state in DTYPES:
        for d_ff, d_model in SHAPES:
            counts = (1, 2, 3, 8, 64)
            reads = ask(*(f"read {io} {state} {d_ff} {d_model} {n} {BIG}" for n in counts))
            assert len({leaf for _, _, leaf, _ in reads}) == 1
            assert all(d_ff <= 1536 and leaf == "8" for direct, _, leaf, _ in reads if direct == "1")
            tokens = ask(*(f"write {io} {state} {d_ff} {d_model} {n} 40 1 {BIG}" for n in counts))
            assert len({(kernel, first, wn) for kernel, first, wn, _ in tokens}) == 1


def test_token_partials_fit_an_owners_workspace(ask):
    """Rows of partial sums per owner: 64 of them, or one per READ chunk."""
    for io, state in DTYPES:
        for d_ff, d_model in SHAPES:
            (kernel, _, wn, _), = ask(f"write {io} {state} {d_ff} {d_model} 3 33 1 {BIG}")
            if kernel == "rows_token":
                assert -(-d_ff // 64) <= TOKEN_ROWS
            elif kernel == "f32" and wn != "1":
                assert -(-d_ff * int(wn) // READ_CHUNK) <= TOKEN_ROWS
            else:
                assert kernel == "stream" or wn == "1"


def test_gemm_deals_every_tile_once(ask):
    sizes = [(c, mt, nt) for c in (1, 2, 8) for mt in (1, 2, 3, 4, 5, 20, 56) for nt in (1, 2, 3, 12, 32, 112)]
    for size, answer in zip(sizes, ask(*(f"gemm {c} {mt} {nt}" for c, mt, nt in sizes))):
        assert answer[0] == "1", size


# below four row tiles or two column tiles of 256 x 128, the smallest that fill
# the XCDs, and one past a multiple of eight tiles
@pytest.mark.parametrize("count,d_ff,d_model", [(8, 256, 4096), (8, 128, 14336), (4, 512, 2048), (8, 768, 768),
                                                (4, 5000, 128), (8, 8192, 64), (1, 256, 1024), (1, 768, 384)])
def test_few_gemm_tiles_reach_every_xcd(ask, count, d_ff, d_model):
    mt, nt = -(-d_ff // 256), -(-d_model // 128)
    (once, *xcds), = ask(f"gemm {count} {mt} {nt}")
    assert once == "1"
    assert max(map(int, xcds)) - min(map(int, xcds)) <= 1


def test_one_launch_read_needs_few_rows_bytes_and_blocks(ask):
    """Both sides of each limit: 1536 rows; 38 MB of state and W0; 1024 blocks of
    32 (bf16 state: 64) columns of one owner, 1536 for bf16 io with fp32 state."""
    one = [("bf16", "f32", 1536, 1032, 4), ("bf16", "f32", 512, 4096, 4), ("bf16", "bf16", 512, 4096, 8),
           ("bf16", "bf16", 128, 14336, 4), ("bf16", "bf16", 8, 4096, 16), ("f32", "f32", 64, 14336, 2),
           ("f32", "bf16", 32, 8192, 8), ("bf16", "f32", 256, 2048, 16), ("bf16", "f32", 8, 8192, 6)]
    two = [("bf16", "f32", 1544, 1032, 4), ("bf16", "f32", 512, 4096, 5), ("f32", "f32", 512, 4096, 4),
           ("bf16", "bf16", 128, 14336, 6), ("bf16", "bf16", 8, 4104, 16), ("bf16", "bf16", 8, 14336, 16),
           ("f32", "f32", 64, 14336, 4), ("f32", "bf16", 8, 14336, 8), ("bf16", "f32", 8, 8200, 6),
           ("bf16", "f32", 8, 1 << 20, 16)]
    for call, direct in [(c, "1") for c in one] + [(c, "0") for c in two]:
        (d, *_), = ask("read " + " ".join(map(str, call)) + f" {BIG}")
        assert d == direct, call


def test_waves_of_a_read_block(ask):
    """Four waves: one owner, and fp32 io with bf16 state past one round of blocks
    whose last column tile is not mostly empty."""
    def waves(*call):
        (direct, w, *_), = ask("read " + " ".join(map(str, call)) + f" {BIG}")
        assert direct == "0"
        return w
    for call in ((9728, 2560, 2), (9728, 2560, 8), (5000, 1528, 5), (3600, 1512, 7), (12000, 1000, 8)):
        assert waves("f32", "bf16", *call) == "4", call
    for call in ((3600, 1512, 1), (5000, 1528, 4), (2048, 2048, 8), (12000, 520, 8), (1536, 4096, 16)):
        assert waves("f32", "bf16", *call) == "8", call
    for io, state in (("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32")):
        assert waves(io, state, 9728, 2560, 1) == "4"
        assert waves(io, state, 9728, 2560, 2) == waves(io, state, 9728, 2560, 8) == "8"


def test_small_bf16_states_without_a_token_stream(ask):
    """bf16 state, C <= 64: the streaming kernel up to one item a CU and for few
    rows (both sides of the lines), and one owner whose blocks fill its slots."""
    def kernel(d_ff, d_model, count, chunk):
        (k, *_), = ask(f"write bf16 bf16 {d_ff} {d_model} {count} {chunk} 0 {BIG}")
        return k
    for small in ((8, 8, 1), (264, 136, 8), (1000, 264, 8), (1024, 1024, 2), (2048, 512, 2), (256, 4096, 2)):
        assert kernel(*small, 1) == kernel(*small, 64) == "stream", small
        assert kernel(*small, 65) == "gemm", small
    for few_rows in ((8, 14336, 32), (32, 14336, 32), (64, 14336, 8), (40, 4096, 32)):
        assert kernel(*few_rows, 1) == kernel(*few_rows, 64) == "stream", few_rows
        assert kernel(*few_rows, 65) == "gemm", few_rows
    for large in ((64, 14336, 16), (72, 14336, 4), (512, 2048, 4), (1024, 1024, 4), (2048, 512, 4), (5000, 128, 1), (8192, 64, 1), (9728, 2560, 2)):
        assert kernel(*large, 1) == kernel(*large, 64) == "gemm", large
    assert kernel(9728, 2560, 1, 16) == kernel(14336, 4096, 1, 16) == "stream"
    assert kernel(9728, 2560, 1, 48) == kernel(14336, 4096, 1, 48) == "gemm"
    assert kernel(10000, 2000, 1, 64) == "stream"


def test_long_chunks_of_fp32_states_by_how_full_the_gemm_runs(ask):
    """Register operands up to 384 ranks, 300 where the GEMM's tiles fill its rounds,
    220 where they fill one; both sides of each line."""
    def kernel(d_ff, d_model, count, chunk):
        (k, *_), = ask(f"write bf16 f32 {d_ff} {d_model} {count} {chunk} 0 {BIG}")
        return k
    for call, last in (((4096, 4096, 1), 220), ((4096, 4096, 3), 300), ((4096, 4096, 8), 300), ((9728, 2560, 1), 384),
                       ((9728, 2560, 3), 384), ((2000, 2000, 3), 384), ((2496, 824, 8), 384), ((8, 8, 1), 384),
                       ((256, 4096, 64), 384), ((1 << 20, 8, 3), 384)):
        assert kernel(*call, 1) == kernel(*call, last) == "rows", call
        assert kernel(*call, last + 1) == "gemm", call
    for call, rows, gemm in (((2000, 2000, 8), 320, 350), ((5000, 1528, 8), 320, 384), ((9728, 2560, 8), 320, 384)):
        assert kernel(*call, rows) == "rows" and kernel(*call, gemm) == "gemm", call


def test_adapter_write_tiles(ask):
    """One tile of 16 evidence rows a block while the blocks fit 256 CUs, whatever
    the chunk and rank; both sides of the line."""
    for call, tiles in (((3, 129, 1, 1), "1"), ((2, 1024, 2, 16), "1"), ((13, 256, 1, 20), "1"), ((2, 128, 16, 32), "1"),
                        ((2, 128, 17, 16), "2"), ((2, 129, 17, 16), "4"), ((2, 129, 17, 17), "2"), ((13, 256, 4, 16), "4"),
                        ((2, 1040, 2, 16), "4"), ((2048, 1024, 64, 32), "2")):
        (got,), = ask("adapter " + " ".join(map(str, call)))
        assert got == tiles, call


def test_the_cache_hint_follows_the_call_and_its_context(ask):
    """The hint is dropped where the context's live states and W0s fit the
    last-level cache and the call is small beside it; never where only one of the
    two holds.  Both sides of both lines."""
    sizes = ((1024, 1024, 1, True), (2000, 2000, 2, True), (3600, 1512, 5, False), (9728, 2560, 2, False))
    for io, state in DTYPES:
        for d_ff, d_model, count, small in sizes:
            for context, fits in ((256000000, True), (256000001, False), (2 * BIG, False)):
                call = f"{io} {state} {d_ff} {d_model} {count}"
                queries = [f"read {call} {context}", f"write {call} 100 0 {context}", f"write {call} 16 1 {context}"]
                for answer in ask(*queries):
                    assert answer[0] == "gemm" or answer[-1] == ("0" if fits and small else "1"), (call, context)
