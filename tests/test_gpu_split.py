"""Step 1 parity: the HIP split kernel against the numpy split, bit for bit, through the C-ABI."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import split
from gpu_util import pack_fp32_fragment_order, pack_fragment_order, to_device

pytestmark = pytest.mark.gpu


def _mode_id(mode):
    import paper_2203_03341_amd as ec
    if isinstance(mode, bool):
        return ec.MODE_BF16_FULL if mode else ec.MODE_FP16_SPLIT
    return {"unscaled": ec.MODE_FP16_UNSCALED, "markidis": ec.MODE_FP16_MARKIDIS, "plain16": ec.MODE_FP16_PLAIN,
            "plainbf": ec.MODE_BF16_PLAIN, "fp32": ec.MODE_FP32_MFMA}[mode]


def _expected(op, store, rows, depth, mode):
    X = store[:rows, :depth] if op == "N" else store[:depth, :rows].T
    X = np.ascontiguousarray(X, dtype=np.float32)
    if mode is True:
        parts = list(split.split_bf16x3(X))
    elif mode is False:
        parts = [p.view(np.uint16) for p in split.split_fp16(X)]
    elif mode in ("unscaled", "markidis"):
        parts = [p.view(np.uint16) for p in split.split_fp16(X, scaled=False)]
    elif mode == "fp32":
        return pack_fp32_fragment_order(X)
    elif mode == "plain16":
        parts = [split.to_fp16_rn(X).view(np.uint16)]
    else:
        parts = [split.to_bf16_rn_bits(X)]
    return pack_fragment_order(parts)


def _run(op, store, rows, depth, mode_bf16, offset_elems=0):
    import torch
    import paper_2203_03341_amd as ec
    mode = _mode_id(mode_bf16)
    h = ec.Handle()
    src = to_device(store)
    nbytes = ec.split_size(rows, depth, mode)
    packed = torch.full((nbytes // 2,), 0x7FFF, dtype=torch.int16, device="cuda")   # poison
    ld = store.shape[0]
    h.split(ec.OP_N if op == "N" else ec.OP_T, rows, depth, src, ld, mode, packed)
    torch.cuda.synchronize()
    got = packed.cpu().numpy().view(np.uint16)
    h.destroy()
    return got


CASES = [
    # (op, rows, depth, ld padding)
    ("N", 256, 256, 0), ("T", 256, 256, 0),
    ("N", 300, 77, 5), ("T", 300, 77, 3),
    ("N", 1, 1, 0), ("T", 1, 1, 0),
    ("N", 33, 1031, 1), ("T", 515, 40, 4), ("T", 70, 129, 1),
    # r-contiguous with a 16-byte aligned leading dimension (the 256-row kernel) and 1, 2, 3 rows past a multiple of 4
    ("N", 301, 77, 3), ("N", 1022, 70, 2), ("N", 515, 40, 1), ("N", 260, 33, 0),
]


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("op,rows,depth,pad", CASES)
def test_split_matches_oracle_bitwise(op, rows, depth, pad, mode_bf16):
    sr, sc = (rows, depth) if op == "N" else (depth, rows)
    for kind in ("urand", "exp15", "exp100"):
        if kind == "urand":
            store = si.urand(sr, sc, seed=1, matrix_id=si.ID_A, ld=sr + pad)
        elif kind == "exp15":
            store = si.exp_rand(sr, sc, -15, 15, seed=2, matrix_id=si.ID_A, ld=sr + pad)
        else:
            store = si.exp_rand(sr, sc, -100, 100, seed=3, matrix_id=si.ID_A, ld=sr + pad)
        got = _run(op, store, rows, depth, mode_bf16)
        want = _expected(op, store, rows, depth, mode_bf16)
        assert got.shape == want.shape
        bad = np.flatnonzero(got != want)
        assert bad.size == 0, (kind, bad[:8], got[bad[:8]], want[bad[:8]])


@pytest.mark.parametrize("mode_bf16", [False, True])
def test_split_edge_values(mode_bf16):
    """Saturation, signed zeros, values that only the scaled residual can hold, FP32 subnormals, Inf, NaN."""
    vals = [0.0, -0.0, 65504.0, 65519.996, 65520.0, 65535.996, -65535.996, 2.0 ** -24, 2.0 ** -25, 2.0 ** -35,
            2.0 ** -36, 1.5 * 2.0 ** -36, 1e-45, -1e-40, 2.0 ** -126, 3.4028234e38, -3.4028234e38, 3.39e38,
            np.inf, -np.inf, 1.0, -1.0, 0.1, 2.0 ** -14, 2.0 ** -15, 1.9999999 * 2.0 ** -15, 6.1e-5, 100000.0, 1e30,
            2.0 ** 116, 2.0 ** 117, -2.0 ** 117, 1e36, -1e38]
    vals = np.array(vals, dtype=np.float32)
    rows, depth = 8, vals.size
    store = np.asfortranarray(np.tile(vals, (rows, 1)) * np.array([[1], [-1], [1], [-1], [1], [-1], [1], [-1]], np.float32))
    store = np.asfortranarray(store.astype(np.float32))
    for op in ("N", "T"):
        st = store if op == "N" else np.asfortranarray(store.T)
        got = _run(op, st, rows, depth, mode_bf16)
        want = _expected(op, st, rows, depth, mode_bf16)
        assert np.array_equal(got, want), np.flatnonzero(got != want)[:10]
    # NaN among ordinary values: where the oracle's parts are NaN the kernel's are (payload bits are not compared), and
    # every other position agrees bit for bit
    mixed = np.asfortranarray(np.tile(np.array([1.0, np.nan, -0.1, 65536.0, np.nan, 3.0e-5, -np.nan, 7.0], np.float32), (6, 1)))
    mixed[2, :] = np.nan
    for op in ("N", "T"):
        st = mixed if op == "N" else np.asfortranarray(mixed.T)
        got = _run(op, st, 6, 8, mode_bf16)
        want = _expected(op, st, 6, 8, mode_bf16)
        if mode_bf16:
            nan_of = lambda bits: ((bits & 0x7F80) == 0x7F80) & ((bits & 0x7F) != 0)
        else:
            nan_of = lambda bits: ((bits & 0x7C00) == 0x7C00) & ((bits & 0x3FF) != 0)
        want_nan = nan_of(want)
        assert want_nan.sum() == (3 if mode_bf16 else 2) * int(np.isnan(mixed).sum())
        assert np.array_equal(nan_of(got), want_nan)
        assert np.array_equal(got[~want_nan], want[~want_nan])


@pytest.mark.parametrize("mode", ["unscaled", "markidis", "plain16", "plainbf", "fp32"])
@pytest.mark.parametrize("op", ["N", "T"])
def test_split_of_comparison_methods(mode, op):
    """Markidis' unscaled residual (Eqs. corr-elm-1, corr-elm-2) and the plain conversions, bit for bit."""
    rows, depth = 300, 77
    sr, sc = (rows, depth) if op == "N" else (depth, rows)
    for store in (si.urand(sr, sc, 4, si.ID_A, ld=sr + 2), si.exp_rand(sr, sc, -20, 15, 5, si.ID_A, ld=sr + 1)):
        got = _run(op, store, rows, depth, mode)
        want = _expected(op, store, rows, depth, mode)
        assert got.shape == want.shape and np.array_equal(got, want)


@pytest.mark.parametrize("mode_bf16", [False, True])
def test_split_of_a_large_operand(mode_bf16):
    """2048 x 3000 in both orientations: every block position of a many-tile grid, bit for bit."""
    for op in ("N", "T"):
        rows, depth = 2048, 3000
        sr, sc = (rows, depth) if op == "N" else (depth, rows)
        store = si.exp_rand(sr, sc, -30, 20, 9, si.ID_B)
        got = _run(op, store, rows, depth, mode_bf16)
        assert np.array_equal(got, _expected(op, store, rows, depth, mode_bf16))


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("rows,depth", [(2048, 4064), (2048, 4096), (2048, 4100), (2040, 4148), (64, 131100)])
def test_split_of_large_operands_with_the_depth_contiguous(mode_bf16, rows, depth):
    """Aligned operands with k contiguous are split four 64 x 32 tiles a block from 1024 such blocks on: one depth below
    that, depths of whole blocks and of one, two and four tiles in the last, a ragged one among them, rows that end
    inside a block; a few values beyond the formats' range.  Bit for bit."""
    store = si.exp_rand(depth, rows, -30, 20, 10, si.ID_B)
    store[depth - 1, rows - 1], store[depth // 2, 3], store[5, rows // 2] = np.inf, 3.39e38, -70000.0
    got = _run("T", store, rows, depth, mode_bf16)
    assert np.array_equal(got, _expected("T", store, rows, depth, mode_bf16))


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("op,rows,depth,pad", [
    ("N", 1021, 4099, 0), ("N", 1022, 4100, 1), ("N", 1023, 4097, 2), ("N", 3, 40, 1), ("N", 2, 33, 2), ("N", 259, 31, 1),
    ("T", 70, 3, 0), ("T", 65, 2, 3), ("T", 67, 1, 3), ("T", 131, 203, 2), ("T", 2047, 4101, 0), ("T", 2046, 4103, 3),
    ("T", 599, 333, 1), ("T", 600, 333, 1), ("T", 399, 6001, 2), ("T", 400, 6001, 2)])
def test_split_of_lines_on_any_alignment(op, rows, depth, pad, mode_bf16):
    """Sources are read 16 bytes at a time wherever their lines start: 0 to 3 values left over at the end of a line, lines
    shorter than one such read, few blocks and many, either side of the row counts from which the XCDs take runs of the
    blocks, in either orientation, NaN behind every line.  Bit for bit."""
    sr, sc = (rows, depth) if op == "N" else (depth, rows)
    store = si.exp_rand(sr, sc, -30, 20, 11, si.ID_A, ld=sr + pad)
    got = _run(op, store, rows, depth, mode_bf16)
    assert np.array_equal(got, _expected(op, store, rows, depth, mode_bf16))


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("op", ["N", "T"])
def test_split_of_lines_on_any_alignment_from_memory_and_from_the_caches(op, mode_bf16):
    """An operand that does not fit the memory-side cache together with its parts is split in other blocks and another
    order than its halves, which do: the packed operand is the packed halves of its rows end to end."""
    import torch
    import paper_2203_03341_amd as ec
    rows, depth = 512, 100003 if mode_bf16 else 131069
    mode = ec.MODE_BF16_FULL if mode_bf16 else ec.MODE_FP16_SPLIT
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    src = torch.randn((depth, rows + 1) if op == "N" else (rows, depth), generator=gen, device="cuda")
    h = ec.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)

    def packed(first, count):
        out = torch.empty(ec.split_size(count, depth, mode), dtype=torch.uint8, device="cuda")
        part = src[:, first:] if op == "N" else src[first:]
        h.split(ec.OP_N if op == "N" else ec.OP_T, count, depth, part, src.shape[1], mode, out)
        return out

    whole, halves = packed(0, rows), [packed(0, 256), packed(256, 256)]
    torch.cuda.synchronize()
    assert torch.equal(whole, torch.cat(halves))
    h.destroy()


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("op", ["N", "T"])
def test_split_of_operands_read_past_the_cache(op, mode_bf16):
    """Aligned operands of 2^26 elements and more with the rows contiguous are read with non-temporal loads.  Row blocks are packed one after the
    other, so the packed operand is the packed halves of its rows end to end, each of them split with ordinary loads
    (which the tests above compare with the oracle)."""
    import torch
    import paper_2203_03341_amd as ec
    rows, depth = 512, (1 << 17) + 4
    mode = ec.MODE_BF16_FULL if mode_bf16 else ec.MODE_FP16_SPLIT
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    src = torch.randn((depth, rows) if op == "N" else (rows, depth), generator=gen, device="cuda")
    h = ec.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)

    def packed(first, count):
        out = torch.empty(ec.split_size(count, depth, mode), dtype=torch.uint8, device="cuda")
        part = src[:, first:] if op == "N" else src[first:]
        h.split(ec.OP_N if op == "N" else ec.OP_T, count, depth, part, src.shape[1], mode, out)
        return out

    whole, halves = packed(0, rows), [packed(0, 256), packed(256, 256)]
    torch.cuda.synchronize()
    assert torch.equal(whole, torch.cat(halves))
    h.destroy()


@pytest.mark.parametrize("mode", ["fp16", "bf16", "markidis", "plain", "fp32"])
@pytest.mark.parametrize("transA,transB,M,N,K", [("T", "N", 8192, 300, 1028), ("T", "N", 2100, 2200, 4132), ("N", "N", 300, 2048, 4128),
                                                 ("T", "T", 2048, 520, 4100), ("T", "N", 2048, 130, 4064), ("T", "N", 8200, 2048, 4096)])
def test_both_operands_in_one_launch_or_two(mode, transA, transB, M, N, K):
    """ecgemm_sgemm splits both operands in one launch while they are small enough, each in blocks of its own variant
    (aligned with k contiguous: of one tile or of four, by size), and ecgemm_split one operand at a time: one of each,
    two of four tiles, one beside the staged variant, depths that end inside a block of four, one pair beyond one launch.
    The product of the operands split one by one has the same bits."""
    import torch
    import paper_2203_03341_amd as ec
    mode = {"fp16": ec.MODE_FP16_SPLIT, "bf16": ec.MODE_BF16_FULL, "markidis": ec.MODE_FP16_MARKIDIS,
            "plain": ec.MODE_FP16_PLAIN, "fp32": ec.MODE_FP32_MFMA}[mode]
    ops = {"N": ec.OP_N, "T": ec.OP_T}
    h = ec.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)
    if mode in (ec.MODE_FP16_SPLIT, ec.MODE_BF16_FULL):
        h.set_shape(ec.SHAPE_128x128_X2)     # (never as one launch on the FP32 operands)
    lda, ldb = M if transA == "N" else K, K if transB == "N" else N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    A, B = torch.randn(M * K, generator=gen, device="cuda"), torch.randn(K * N, generator=gen, device="cuda")
    whole, parts = torch.full((N, M), float("nan"), device="cuda"), torch.full((N, M), float("nan"), device="cuda")
    h.sgemm(ops[transA], ops[transB], M, N, K, 1.0, A, lda, B, ldb, 0.0, whole, M, mode)
    packed_a = torch.empty(ec.split_size(M, K, mode), dtype=torch.uint8, device="cuda")
    packed_b = torch.empty(ec.split_size(N, K, mode), dtype=torch.uint8, device="cuda")
    h.split(ops[transA], M, K, A, lda, mode, packed_a)
    h.split(ec.OP_T if transB == "N" else ec.OP_N, N, K, B, ldb, mode, packed_b)
    h.product(M, N, K, 1.0, packed_a, packed_b, 0.0, parts, M, mode)
    torch.cuda.synchronize()
    assert not bool(torch.isnan(whole).any())
    assert torch.equal(whole, parts)
    h.destroy()


def test_a_leading_dimension_off_the_cache_lines_is_not_fetched_twice():
    """The same large operand with the depth contiguous, its rows on whole cache lines (leading dimension 9024) and not
    (9000, still a multiple of 16 bytes): neighbouring blocks share lines in the second, which one of them then finds in a
    cache (118 us against 117; 167 with loads that went past the caches)."""
    import torch
    import paper_2203_03341_amd as ec
    rows = depth = 9000
    h = ec.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)
    src = torch.rand(rows * 9024, device="cuda")
    packed = torch.empty(ec.split_size(rows, depth, ec.MODE_FP16_SPLIT), dtype=torch.uint8, device="cuda")

    def best_us(ld):
        def timed():
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                h.split(ec.OP_T, rows, depth, src, ld, ec.MODE_FP16_SPLIT, packed)
            stop.record()
            torch.cuda.synchronize()
            return start.elapsed_time(stop) * 1e3 / 20
        return min(timed() for _ in range(6))

    best_us(9024)
    whole, shared = best_us(9024), best_us(9000)
    assert shared < 1.2 * whole, (whole, shared)
    h.destroy()


@pytest.mark.parametrize("mode_bf16", [False, True])
@pytest.mark.parametrize("transA,transB,M,N,K,pad", [("N", "T", 1030, 1101, 900, 1),     # rows contiguous, few tiles together: 64 rows a block
                                                     ("N", "T", 2050, 1999, 900, 1),     # many: 256
                                                     ("N", "T", 1028, 333, 201, 0),      # on 16 bytes beside lines that are not
                                                     ("T", "T", 131, 1027, 333, 2),      # beside the depth contiguous
                                                     ("N", "N", 2059, 2111, 1500, 3)])   # four tiles a block beside 256 rows
def test_two_operands_split_together_are_what_each_is_alone(transA, transB, M, N, K, pad, mode_bf16):
    """The operands of a product are split in one launch, in blocks that depend on both: the product has the bits of one
    made from operands that were split one by one, in other blocks.  NaN behind every line."""
    import torch
    import paper_2203_03341_amd as ec
    mode = ec.MODE_BF16_FULL if mode_bf16 else ec.MODE_FP16_SPLIT
    ops = {"N": ec.OP_N, "T": ec.OP_T}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)

    def operand(cols, rows):
        store = torch.full((cols, rows + pad), float("nan"), device="cuda")
        store[:, :rows] = torch.randn((cols, rows), generator=gen, device="cuda")
        return store

    A = operand(*((K, M) if transA == "N" else (M, K)))
    B = operand(*((N, K) if transB == "N" else (K, N)))
    h = ec.Handle()
    h.set_stream(torch.cuda.current_stream().cuda_stream)
    h.set_shape(ec.SHAPE_128x128_X2)
    together, alone = torch.zeros((N, M), device="cuda"), torch.zeros((N, M), device="cuda")
    h.sgemm(ops[transA], ops[transB], M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, together, M, mode)
    packed = [torch.empty(ec.split_size(rows, K, mode), dtype=torch.uint8, device="cuda") for rows in (M, N)]
    h.split(ops[transA], M, K, A, A.shape[1], mode, packed[0])
    h.split(ec.OP_T if transB == "N" else ec.OP_N, N, K, B, B.shape[1], mode, packed[1])
    h.product(M, N, K, 1.0, packed[0], packed[1], 0.0, alone, M, mode)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(alone).all()) and torch.equal(together, alone)
    h.destroy()
