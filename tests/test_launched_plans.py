"""What the GEMM entry points launch, against what gemm_plan says (CPU only): the C ABI and
the selector built host-only with tests/record_stub.cpp in place of the device side."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2512_13282_amd import binding as b

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2512_13282_amd", "csrc")
I8, BF = b.GEMM_DTYPE_I8_I32, b.GEMM_DTYPE_BF16_F32
FA, FB, FC = 1 << 40, 1 << 41, 3 << 40    # 16-byte aligned addresses, far apart (never dereferenced)
FIELDS = ("config", "split_k", "k_chunk", "reduce", "grid", "epilogue", "static_scratch", "tiles")


class Recorder:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        self.lib.gemm_plan.argtypes = self.lib.gemm_plan_bt.argtypes = b.lib().gemm_plan.argtypes

    def call(self, name, M, N, K, bt, a_off=0):
        fn = getattr(self.lib, name + ("_bt" if bt else ""))
        i64, p = ctypes.c_int64, ctypes.c_void_p
        shift = [4] if name in ("gemm_i8_i8", "gemm_i8_i16") else []
        fn.argtypes = [i64, i64, i64, p, i64, p, i64, p, i64] + [ctypes.c_int] * len(shift) + [p]
        rc = fn(M, N, K, FA + a_off, max(K, 1), FB, max(K if bt else N, 1), FC, max(N, 1), *shift, None)
        out = (i64 * 8)()
        self.lib.recorded_launch(out)
        return rc, dict(zip(FIELDS, out))

    def plan(self, dtype, M, N, K, bt, a_off=0):
        info = b.PlanInfo()
        fn = self.lib.gemm_plan_bt if bt else self.lib.gemm_plan
        rc = fn(dtype, M, N, K, max(K, 1), max(K if bt else N, 1), max(N, 1), FA + a_off, FB, FC, ctypes.byref(info))
        assert rc == b.GEMM_OK
        return info


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rec") / "libgemm_rec.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    os.path.join(CSRC, "gemm_api.cpp"), os.path.join(CSRC, "selector.cpp"),
                    os.path.join(HERE, "record_stub.cpp"), "-o", out], check=True, capture_output=True, text=True)
    return Recorder(out)


def _shapes(n, seed):
    rng = random.Random(seed)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    for _ in range(n):
        M, N, K = log(1, 8192), log(32, 14336), log(32, 14336)
        if rng.random() < 0.7:
            N, K = max(64, N // 64 * 64), max(64, K // 64 * 64)
        yield M, N, K, rng.randint(0, 1)


SAME = ("config", "split_k", "k_chunk", "grid")
ATOMIC = (b.GEMM_REDUCE_ATOMIC, b.GEMM_REDUCE_ATOMIC_FLAG)


def test_bf16_plans_do_not_depend_on_the_output_type(rec):
    """gemm_bf16_bf16 runs the tile, K slices and reduction of gemm_bf16_f32, which are what
    gemm_plan reports: the fp32 sums that it rounds are that call's."""
    known = [(192, 1984, 2624, 1), (3424, 128, 7680, 0), (589, 771, 1647, 1), (128, 704, 6272, 1)]
    for M, N, K, bt in known + list(_shapes(300, 1)):
        p = rec.plan(BF, M, N, K, bt)
        for name in ("gemm_bf16_f32", "gemm_bf16_bf16"):
            rc, x = rec.call(name, M, N, K, bt)
            assert rc == b.GEMM_OK and [x[k] for k in SAME] == [p.config, p.split_k, p.k_chunk, p.grid], (name, M, N, K)
            assert x["split_k"] == 1 or x["reduce"] == p.reduce_in_kernel


def test_narrowed_int8_plans(rec):
    """gemm_i8_i32 runs what gemm_plan reports.  The narrowed calls run measured and forced plans
    too, and plans of their own elsewhere; none adds K slices into C."""
    tuned = [(16, 4096, 14336, 0), (2048, 4096, 11008, 1), (48, 14336, 4096, 1), (64, 4096, 14336, 1)]
    for M, N, K, bt in tuned + list(_shapes(300, 4)):
        p = rec.plan(I8, M, N, K, bt)
        rc, w = rec.call("gemm_i8_i32", M, N, K, bt)
        assert rc == b.GEMM_OK and [w[k] for k in SAME] == [p.config, p.split_k, p.k_chunk, p.grid]
        for name in ("gemm_i8_i8", "gemm_i8_i16"):
            rc, x = rec.call(name, M, N, K, bt)
            assert rc == b.GEMM_OK and (x["split_k"] == 1 or x["reduce"] not in ATOMIC), (name, M, N, K, bt, x)
            if (M, N, K, bt) in tuned:
                assert p.source != b.GEMM_PLAN_FROM_MODEL and [x[k] for k in SAME] == [w[k] for k in SAME]
    for reduce in ATOMIC:
        rec.lib.gemm_force_plan(I8, b.GEMM_KERNEL_AUTO, 28, 4)
        rec.lib.gemm_force_reduce(I8, reduce)
        try:
            assert rec.call("gemm_i8_i32", 16, 4096, 14336, 0)[1]["reduce"] == reduce
            rc, x = rec.call("gemm_i8_i8", 16, 4096, 14336, 0)
            assert rc == b.GEMM_OK and (x["config"], x["split_k"], x["reduce"]) == (28, 4, b.GEMM_REDUCE_SEPARATE)
        finally:
            rec.lib.gemm_force_reduce(I8, -1)
            rec.lib.gemm_force_plan(I8, b.GEMM_KERNEL_AUTO, -1, 0)


@pytest.mark.parametrize("M,N,K,bt", [(12, 1024, 320, 1), (16, 64, 384, 1), (3, 64, 512, 0), (50, 3712, 512, 1),
                                      (2431, 64, 640, 0), (2697, 128, 1152, 1)])
def test_small_narrowed_int8_calls_run_whole(rec, M, N, K, bt):
    """Calls of 4-6 us whose int32 form splits K for the price of adding into C: the kernel that
    sums a narrowed call's slices would cost them half as much again."""
    for name in ("gemm_i8_i8", "gemm_i8_i16"):
        rc, x = rec.call(name, M, N, K, bt)
        assert rc == b.GEMM_OK and x["split_k"] == 1, x


LIMIT = (16 << 20) - (64 << 10)


def test_noalloc_runs_the_best_plan_that_fits(rec):
    """gemm_bf16_f32_noalloc runs gemm_bf16_f32's plan where its partials fit the fixed scratch,
    else one chosen with the scratch as a bound: not the tile of the split plan on the few
    compute units that it fills unsplit."""
    changed = 0
    for M, N, K, _ in list(_shapes(400, 2)):
        p = rec.plan(BF, M, N, K, 0)
        rc, x = rec.call("gemm_bf16_f32_noalloc", M, N, K, 0)
        assert rc == b.GEMM_OK and x["static_scratch"] == 1
        planes = x["split_k"] * M * N * 4 if x["split_k"] > 1 else 0
        assert planes <= LIMIT and (x["reduce"] != b.GEMM_REDUCE_LAST_SLICE or x["tiles"] * 4 <= 64 << 10)
        if p.workspace_bytes <= LIMIT:
            assert [x[k] for k in ("config", "split_k", "k_chunk")] == [p.config, p.split_k, p.k_chunk]
        else:
            changed += 1
    assert changed >= 5


@pytest.mark.parametrize("M,N,K", [(1520, 1856, 6976), (196, 2833, 7273), (330, 2555, 9583), (1200, 1792, 3136),
                                   (512, 8192, 8192), (2048, 4096, 14336), (256, 13824, 5120)])
def test_noalloc_fallback_fills_the_chip(rec, M, N, K):
    """Calls whose split plan does not fit: 23 to 128 workgroups if that plan's tile ran
    unsplit, on 256 compute units (1.1-3.8 times the time of the plans below)."""
    assert rec.plan(BF, M, N, K, 0).workspace_bytes > LIMIT
    rc, x = rec.call("gemm_bf16_f32_noalloc", M, N, K, 0)
    assert rc == b.GEMM_OK and x["grid"] >= 130, x
