"""The any-alignment tile kernels (GENERIC) where their 16-byte loads can go wrong,
through the C ABI (needs an MI355X): rows of 16 bytes (the shortest they take) and one
element less (the element-wise kernel) or more, K and N one past and one short of a
stage, a piece and a tile, odd row pitches, operands starting at an odd element, K
split so that only the last slice holds a ragged end, and non-finite values in the
memory between and after the rows, which no stored result may see.  int8 against the
oracle bit for bit; bf16 on integer-valued operands, whose fp32 sums are exact in any
order, so equality is required there too.
"""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_13282_amd import binding as b
from paper_2512_13282_amd import inputs
import gpu_helpers as g

pytestmark = pytest.mark.gpu
I8, BF = g.I8, g.BF
CONFIGS = [0, 1, 41, 42, 43]


@pytest.fixture(autouse=True)
def _reset_plan():
    g.unforce()
    yield
    g.unforce()


def _dev(x, pad, off):
    """x on the GPU with `pad` elements between rows and `off` before the first; what is not
    the matrix is NaN (bf16) or -128, 64 elements after the last row too."""
    rows, cols = x.shape
    host = x.view(np.int16) if x.dtype == np.uint16 else x
    fill = np.array(0x7FC1 if x.dtype == np.uint16 else -128).astype(host.dtype)
    ld = cols + pad
    flat = np.full(off + (rows - 1) * ld + cols + 64, fill, dtype=host.dtype)
    np.lib.stride_tricks.as_strided(flat[off:], (rows, cols), (ld * host.itemsize, host.itemsize))[:] = host
    return torch.from_numpy(flat).to(g.DEV), ld


def _check(dtype, M, N, K, bt, pad, off, seed):
    if dtype == I8:
        A, B = inputs.make_inputs("int8", M, N, K, seed=seed)
        ref, ovf = oracle.get().gemm_i8_i32(A, B)
        assert ovf == 0
    else:
        A = inputs.small_int_bf16_matrix(M, K, seed=seed)
        B = inputs.small_int_bf16_matrix(K, N, seed=seed + 1)
        ref = oracle.get().gemm_bf16_f64(A, B)
    e = 1 if dtype == I8 else 2
    dA, lda = _dev(A, pad[0], off[0])
    dB, ldb = _dev(np.ascontiguousarray(B.T) if bt else B, pad[1], off[1])
    dC, ldc = g.out_buffer(M, N, dtype, pad[2])
    names = (("gemm_i8_i32", "gemm_i8_i32_bt"), ("gemm_bf16_f32", "gemm_bf16_f32_bt"))
    rc = getattr(b, names[dtype][bt])(M, N, K, dA.data_ptr() + off[0] * e, lda, dB.data_ptr() + off[1] * e, ldb,
                                      dC.data_ptr(), ldc, torch.cuda.current_stream().cuda_stream)
    assert rc == b.GEMM_OK, b.gemm_status_string(rc)
    torch.cuda.synchronize()
    C = dC.cpu().numpy()[: M * ldc].reshape(M, ldc)[:, :N]
    assert np.array_equal(C.astype(np.float64), ref.astype(np.float64))


@pytest.mark.parametrize("bt", [0, 1], ids=["row", "col"])
@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("dtype", [I8, BF], ids=["i8", "bf16"])
def test_edges(dtype, config, bt):
    piece = 16 if dtype == I8 else 8
    stage = 8 * piece
    shapes = [(1, piece, piece), (5, piece + 1, 3 * piece - 1), (33, 2 * piece - 1, stage), (63, 129, stage + 1),
              (130, 257, 2 * stage - 1), (257, 131, 3 * stage + piece + 3), (260, 300, 5 * stage + 1)]
    if config < 2:                                        # the element-wise kernel beside it
        shapes += [(3, piece - 1, piece + 1), (40, piece + 9, piece - 1)]
    for i, (M, N, K) in enumerate(shapes):
        for split in (1, 3):
            g.force(dtype, b.GEMM_KERNEL_AUTO, config, split)
            for pad, off in (((0, 0, 0), (0, 0)), ((1, 3, 1), (1, 1)), ((0, 5, 0), (3, 0))):
                print(f"dtype={dtype} config={config} bt={bt} {(M, N, K)} split={split} pad={pad} off={off}", flush=True)
                _check(dtype, M, N, K, bt, pad, off, seed=500 + i)


@pytest.mark.parametrize("bt", [0, 1], ids=["row", "col"])
@pytest.mark.parametrize("dtype", [I8, BF], ids=["i8", "bf16"])
def test_selected_plans(dtype, bt):
    """The selector's own choice over rows and depths, odd sizes."""
    for i, (M, N, K) in enumerate([(1, 1031, 2053), (9, 2049, 1025), (50, 515, 4099), (200, 1001, 777), (1023, 771, 519),
                                   (3001, 65, 147), (777, 2051, 33)]):
        print(f"dtype={dtype} bt={bt} {(M, N, K)}", flush=True)
        _check(dtype, M, N, K, bt, (0, 0, 0), (0, 0), seed=600 + i)
