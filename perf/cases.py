"""The GEMM calls whose speed is followed: what they are, their inputs and exact results.

Every case is one call through the Python binding, as a program that serves or trains a
network makes it: operands and the output buffer are on the GPU, the call is queued on the
current stream, nothing waits.  int32 / fp32 results go through the torch helpers, narrowed
results through the entry points that take addresses.
"""
import math

import torch

from paper_2512_13282_amd import binding


def _case(name, dtype, M, N, K, layout="row", out="wide", pad=0):
    """C (M x N) = A (M x K) . B (K x N).  layout: how B is stored, "row" (K x N) or "col"
    (N x K, a linear layer's weight).  out: "wide" (int32 / fp32), or "bf16", "i8", "i16".
    pad: extra elements in each row of A's buffer (A is a slice of a wider activation)."""
    c = {"dtype": dtype, "M": M, "N": N, "K": K, "layout": layout, "out": out, "pad": pad}
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest call in use: a tile-sized product where the launch is what counts.
        _case("i8_256_cube", "i8", 256, 256, 256),
        # A small dense layer.
        _case("bf16_1024_cube", "bf16", 1024, 1024, 1024),
        # One token through a feed-forward weight stored N x K: a read of B.
        _case("bf16_decode_m1", "bf16", 1, 14336, 4096, "col"),
        # A small decode batch through a down projection.
        _case("i8_decode_m16", "i8", 16, 4096, 14336),
        # A decode batch of a size that is no power of two, activations kept in bf16.
        _case("bf16_decode_m48", "bf16", 48, 11008, 4096, "col", "bf16"),
        # Prefill of 2048 tokens, up projection, activations kept in bf16.
        _case("bf16_prefill_up", "bf16", 2048, 11008, 4096, "col", "bf16"),
        # Prefill, down projection, quantised network: int8 activations out.
        _case("i8_prefill_down", "i8", 2048, 4096, 11008, "col", "i8"),
        # The headline products.
        _case("i8_8192_cube", "i8", 8192, 8192, 8192),
        _case("bf16_8192_cube", "bf16", 8192, 8192, 8192),
        # The head over a vocabulary of odd size: rows of B start at any even address.
        _case("bf16_head_odd", "bf16", 256, 32003, 4096),
        # A first convolution as a product over gathered 7 x 7 x 3 patches of four images.
        _case("i8_patches_k147", "i8", 50176, 64, 147),
        # A layer with odd sizes throughout.
        _case("bf16_odd_layer", "bf16", 2047, 2051, 2049, "col", "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "prefill", "dense", "patches"])
    if kind == "decode":        # up to 64 rows through a projection
        M, N, K = _log_int(rng, 1, 64), _log_int(rng, 1024, 14336), _log_int(rng, 1024, 14336)
    elif kind == "prefill":     # a prompt, or a chunk of one, through a projection
        M, N, K = _log_int(rng, 65, 2048), _log_int(rng, 1024, 14336), _log_int(rng, 1024, 14336)
    elif kind == "dense":       # any dense product
        M, N, K = (_log_int(rng, 128, 8192) for _ in range(3))
    else:                       # a convolution over gathered patches
        M, N, K = _log_int(rng, 3136, 65536), _log_int(rng, 32, 512), _log_int(rng, 27, 1152)
    if rng.random() < 0.6:      # sizes as most networks have them; the rest are any number
        N, K = max(64, N // 64 * 64), max(64, K // 64 * 64)
        if M > 64:
            M = M // 16 * 16
    else:                       # odd rows too
        N, K = (x + 1 if rng.random() < 0.5 and x % 2 == 0 else x for x in (N, K))
    most = 1 << 36              # no drawn case is larger than a 4096 cube
    if M * N * K > most:
        M = max(65, most // (N * K))
    dtype = rng.choice(["bf16", "i8"])
    out = rng.choice(["wide", "wide", "bf16"] if dtype == "bf16" else ["wide", "wide", "i8", "i16"])
    pad = rng.choice([0, 0, 0, 64])
    return _case(None, dtype, M, N, K, rng.choice(["row", "col"]), out, pad)


def _shift(case):
    """The power of two that a narrowed int8 result is divided by: results then spread over
    a quarter of the output's range on either side (inputs have a spread of 32)."""
    spread = 32.0 * 32.0 * math.sqrt(case["K"])
    return max(0, round(math.log2(spread / (32.0 if case["out"] == "i8" else 8192.0))))


def _operands(case, seed):
    M, N, K, pad = case["M"], case["N"], case["K"], case["pad"]
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    rows, cols = (K, N) if case["layout"] == "row" else (N, K)
    if case["dtype"] == "bf16":     # activations of unit spread, weights of a trained layer's
        A = torch.randn(M, K + pad, device=dev, generator=gen).to(torch.bfloat16)
        B = (torch.randn(rows, cols, device=dev, generator=gen) * 0.02).to(torch.bfloat16)
    else:                           # quantised to four standard deviations
        A = (torch.randn(M, K + pad, device=dev, generator=gen) * 32).round_().clamp_(-127, 127).to(torch.int8)
        B = (torch.randn(rows, cols, device=dev, generator=gen) * 32).round_().clamp_(-127, 127).to(torch.int8)
    return A[:, :K], B


_OUT = {("bf16", "wide"): torch.float32, ("bf16", "bf16"): torch.bfloat16,
        ("i8", "wide"): torch.int32, ("i8", "i8"): torch.int8, ("i8", "i16"): torch.int16}
_WIDE = {"bf16": binding.mm_bf16_f32, "i8": binding.mm_i8_i32}
_NARROW = {("bf16", "row"): binding.gemm_bf16_bf16, ("bf16", "col"): binding.gemm_bf16_bf16_bt,
           ("i8", "row"): binding.gemm_i8_i8, ("i8", "col"): binding.gemm_i8_i8_bt,
           ("i16", "row"): binding.gemm_i8_i16, ("i16", "col"): binding.gemm_i8_i16_bt}


def prepare(case, seed):
    A, B = _operands(case, seed)
    C = torch.empty(case["M"], case["N"], dtype=_OUT[case["dtype"], case["out"]], device=A.device)
    return {"case": case, "A": A, "B": B if case["layout"] == "row" else B.t(), "stored_B": B, "C": C,
            "shift": _shift(case)}


def run(state):
    case, A, C = state["case"], state["A"], state["C"]
    if case["out"] == "wide":
        return _WIDE[case["dtype"]](A, state["B"], out=C)
    B = state["stored_B"]
    args = (case["M"], case["N"], case["K"], A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0),
            C.data_ptr(), C.stride(0))
    if case["dtype"] == "i8":
        args += (state["shift"],)
    rc = _NARROW[case["out"], case["layout"]](*args, torch.cuda.current_stream().cuda_stream)
    if rc != binding.GEMM_OK:
        raise binding.GemmError(rc)
    return C


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    e = 2 if case["dtype"] == "bf16" else 1
    o = _OUT[case["dtype"], case["out"]].itemsize
    return {"bytes": M * K * e + K * N * e + M * N * o, "flops": 2 * M * N * K}


def tolerance(case):
    if case["dtype"] == "i8":
        return "exact"
    if case["out"] == "wide":
        # Against 64 bits the sums are 2e-7 to 6e-7 off (K = 1024 to 8192); two orders of summing
        # differ by as much again.
        return {"rel": 3e-6, "max": 3e-5}
    # The same sums rounded to bf16: a few in ten thousand results fall on the other side of a
    # rounding boundary, each by one step (up to 1/128 of its value).
    return {"rel": 2e-4, "max": 0.01}


def exact(case, seed):
    A, B = _operands(case, seed)
    if case["layout"] == "col":
        B = B.t().contiguous()
    C = torch.empty(case["M"], case["N"], dtype=torch.float64, device=A.device)
    wide_b = B.double()
    for r in range(0, case["M"], 8192):     # int8 sums stay far below 2^53: exact in fp64 too
        torch.mm(A[r:r + 8192].double(), wide_b, out=C[r:r + 8192])
    if case["dtype"] == "bf16":
        return C
    if case["out"] == "wide":
        return C.to(torch.int32)
    top = 127 if case["out"] == "i8" else 32767
    C = torch.round(C / 2.0 ** _shift(case)).clamp_(-top - 1, top)      # ties to even
    return C.to(_OUT[case["dtype"], case["out"]])
