"""The calls whose speed matters to a user of the library, from the smallest to the largest, as plain data plus the few
lines a program writes around them.

Matrices are column-major, as the C interface takes them: a `rows` x `cols` matrix with leading dimension `ld` is a
float32 tensor of shape (cols, ld).  Every program here holds what such a program keeps between calls: a handle on its
stream, a workspace of the size the library asks for, and its matrices.
"""
import math

import torch

import paper_2203_03341_amd as ec

_MODES = {"fp16": ec.MODE_FP16_SPLIT, "bf16": ec.MODE_BF16_FULL, "auto": ec.MODE_AUTO}
_OPS = {"N": ec.OP_N, "T": ec.OP_T}
_LARGEST_FLOPS = 3 * 2.0 * 16384 ** 3


def _case(call, mode, M, N, K, trans="NN", pad=0, alpha=1.0, beta=0.0, inputs="uniform"):
    return {"call": call, "mode": mode, "M": M, "N": N, "K": K, "trans": trans, "pad": pad, "alpha": alpha, "beta": beta,
            "inputs": inputs}


def listed():
    def named(name, *args, **more):
        return dict(_case(*args, **more), name=name)

    return [
        # one small product among many (a block of a blocked solver, a small layer): launches and latency
        named("small_256_fp16", "sgemm", "fp16", 256, 256, 256),
        # the same with nothing even about it: odd sizes, padded leading dimensions, both operands transposed, alpha
        named("small_ragged_bf16", "sgemm", "bf16", 300, 200, 77, trans="TT", pad=3, alpha=1.5),
        # a small product whose caller knows nothing of its inputs' exponents and leaves the mode to the library
        named("auto_1024", "sgemm", "auto", 1024, 1024, 1024),
        # ordinary sizes: a few hundred output tiles, so that the chip is just about filled
        named("square_2048_fp16", "sgemm", "fp16", 2048, 2048, 2048, trans="NT"),
        named("square_4096_fp16", "sgemm", "fp16", 4096, 4096, 4096),
        # the size the method's throughput is quoted at, exponents over the whole window of the FP16 pair
        named("square_16384_fp16", "sgemm", "fp16", 16384, 16384, 16384, inputs="window"),
        # full exponent range, C updated in place with alpha and beta (a trailing update, a residual)
        named("square_8192_bf16_update", "sgemm", "bf16", 8192, 8192, 8192, alpha=1.5, beta=0.5, inputs="wide"),
        # the same inputs with the mode left to the library, which runs them as FP16 on scaled rows and columns
        named("auto_8192_wide", "sgemm", "auto", 8192, 8192, 8192, alpha=1.5, beta=0.5, inputs="wide"),
        # shallow: a rank-256 product of two tall panels, half of whose time is writing C
        named("shallow_16384x256_fp16", "sgemm", "fp16", 16384, 16384, 256),
        # deep: a Gram matrix of long vectors, where reading A and B counts as much as multiplying them
        named("deep_1024x65536_fp16", "sgemm", "fp16", 1024, 1024, 65536),
        # large with odd sizes, rows that start on no particular alignment
        named("odd_4095_bf16", "sgemm", "bf16", 4095, 3001, 5003, trans="TN"),
        # one operand split once and kept for many products: split the other one, then multiply
        named("kept_512x4096_fp16", "kept", "fp16", 512, 4096, 4096, trans="TN"),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call, mode = rng.choice([("sgemm", "fp16"), ("sgemm", "fp16"), ("sgemm", "fp16"), ("sgemm", "bf16"), ("sgemm", "bf16"),
                             ("sgemm", "auto"), ("kept", "fp16"), ("kept", "bf16")])
    while True:
        M, N, K = _log_uniform(rng, 64, 16384), _log_uniform(rng, 64, 16384), _log_uniform(rng, 64, 65536)
        if rng.random() < 0.5:      # half of all programs have round sizes
            M, N, K = (max(64, (v + 32) // 64 * 64) for v in (M, N, K))
        if 6 * 2.0 * M * N * K <= 0.25 * _LARGEST_FLOPS and (M + N) * K <= 2 ** 28:
            break
    update = call == "sgemm" and rng.random() < 0.3
    inputs = rng.choice(["uniform", "wide"]) if mode == "auto" else rng.choice(["uniform", "window"])
    return _case(call, mode, M, N, K, trans=rng.choice(["NN", "NT", "TN", "TT"]), pad=rng.choice([0, 0, 0, 1, 3, 4]),
                 alpha=1.5 if update else 1.0, beta=0.5 if update else 0.0, inputs=inputs)


def _uniform(cols, ld, gen):
    """uniform(-1, 1) with a full 24-bit significand in every binade"""
    out = torch.empty((cols, ld), dtype=torch.float32, device="cuda")
    step = max(1, (1 << 26) // ld)
    for at in range(0, cols, step):
        part = out[at:at + step]
        part.copy_(torch.rand(part.shape, generator=gen, device="cuda", dtype=torch.float64) * 2.0 - 1.0)
    return out


def _exponents(cols, ld, lo, hi, gen):
    """sign * (1 + u) * 2^e, e uniform in lo .. hi"""
    out = torch.empty((cols, ld), dtype=torch.int32, device="cuda")
    step = max(1, (1 << 26) // ld)
    for at in range(0, cols, step):
        part = out[at:at + step]
        bits = torch.randint(0, 1 << 23, part.shape, generator=gen, device="cuda", dtype=torch.int32)
        bits |= (torch.randint(lo, hi + 1, part.shape, generator=gen, device="cuda", dtype=torch.int32) + 127) << 23
        sign = torch.randint(0, 2, part.shape, generator=gen, device="cuda", dtype=torch.int32) << 31
        part.copy_(bits | sign)
    return out.view(torch.float32)


def _inputs(case, seed):
    """A, B and, for an update, the C it starts from, as the program stores them"""
    M, N, K, pad = case["M"], case["N"], case["K"], case["pad"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def matrix(cols, ld, window, wide):
        if case["inputs"] == "uniform":
            return _uniform(cols, ld, gen)
        return _exponents(cols, ld, *(window if case["inputs"] == "window" else wide), gen)

    a_rows, a_cols = (M, K) if case["trans"][0] == "N" else (K, M)
    b_rows, b_cols = (K, N) if case["trans"][1] == "N" else (N, K)
    A = matrix(a_cols, a_rows + pad, (-15, 15), (-100, 100))
    B = matrix(b_cols, b_rows + pad, (-15, 15), (-15, 14))
    return A, B, _uniform(N, M + pad, gen) if case["beta"] != 0.0 else None


def prepare(case, seed):
    M, N, K, pad, mode = case["M"], case["N"], case["K"], case["pad"], _MODES[case["mode"]]
    trans_a, trans_b = _OPS[case["trans"][0]], _OPS[case["trans"][1]]
    A, B, C_in = _inputs(case, seed)
    s = {"case": case, "M": M, "N": N, "K": K, "mode": mode, "trans_a": trans_a, "trans_b": trans_b,
         "lda": A.shape[1], "ldb": B.shape[1], "ldc": M + pad, "A": A, "B": B,
         "C": torch.zeros((N, M + pad), dtype=torch.float32, device="cuda")}
    if C_in is not None:
        s["C_in"] = C_in
    handle = ec.Handle()
    handle.set_stream(torch.cuda.current_stream().cuda_stream)
    nbytes = max(256, handle.workspace_size(trans_a, trans_b, M, N, K, mode))
    s["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    handle.set_workspace(s["workspace"], nbytes)
    s["handle"] = handle
    if case["call"] == "kept":
        s["packed_a"] = torch.empty(ec.split_size(M, K, mode), dtype=torch.uint8, device="cuda")
        s["packed_b"] = torch.empty(ec.split_size(N, K, mode), dtype=torch.uint8, device="cuda")
        handle.split(ec.OP_T if trans_b == ec.OP_N else ec.OP_N, N, K, s["B"], s["ldb"], mode, s["packed_b"])
    return s


def run(s):
    case, h = s["case"], s["handle"]
    if case["call"] == "kept":
        h.split(s["trans_a"], s["M"], s["K"], s["A"], s["lda"], s["mode"], s["packed_a"])
        h.product(s["M"], s["N"], s["K"], case["alpha"], s["packed_a"], s["packed_b"], case["beta"], s["C"], s["ldc"], s["mode"])
    else:
        if case["beta"] != 0.0:     # an update starts from the C that the program has at that point
            s["C"].copy_(s["C_in"])
        h.sgemm(s["trans_a"], s["trans_b"], s["M"], s["N"], s["K"], case["alpha"], s["A"], s["lda"], s["B"], s["ldb"],
                case["beta"], s["C"], s["ldc"], s["mode"])
    return s["C"][:, :s["M"]]


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    # three FP16 products, six BF16 products; the automatic mode's choice for these inputs is an FP16 arrangement
    products = 6 if case["mode"] == "bf16" else 3
    bytes_a, bytes_b, bytes_c = 4 * M * K, 4 * K * N, 4 * M * N
    if case["call"] == "kept":      # the kept operand is read as it is kept: two FP16 or three BF16 parts per value
        bytes_b = (6 if case["mode"] == "bf16" else 4) * K * N
    return {"bytes": bytes_a + bytes_b + bytes_c * (2 if case["beta"] != 0.0 else 1), "flops": products * 2.0 * M * N * K}


def tolerance(case):
    # Measured against a product in 64 bits: 1.2e-7 at K = 256 up to 8.2e-7 at K = 16384 (the FP32 sum of the matrix
    # unit, growing with the square root of the depth it runs over), 5.8e-7 for 65536 deep in slices.  Four times that.
    return {"rel": 4.0 * (1.2e-7 + 5.5e-9 * math.sqrt(min(case["K"], 16384)))}


def exact(case, seed):
    """The same product in 64 bits, rounded nowhere, laid out as `run` returns it"""
    M, N, pad = case["M"], case["N"], case["pad"]
    A, B, C_in = _inputs(case, seed)

    C_in = None if C_in is None else C_in[:, :M]

    def logical(X, trans):      # (cols, ld) as stored -> op(X) as a row-major matrix
        X = X[:, :X.shape[1] - pad]
        return X.t() if trans == "N" else X

    A, B = logical(A, case["trans"][0]), logical(B, case["trans"][1]).double()
    out = torch.empty((N, M), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // case["K"])     # rows of A at a time
    for at in range(0, M, step):
        rows = case["alpha"] * (A[at:at + step].double() @ B)
        if C_in is not None:
            rows += case["beta"] * C_in[:, at:at + step].t().double()
        out[:, at:at + step] = rows.t()
    return out
