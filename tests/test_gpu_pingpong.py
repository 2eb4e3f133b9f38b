"""The ping-pong kernel (configuration 44, and 13 for row-major B) and the narrow kernel with
three stages (45) where their schedules, and the quadrant layout, can go wrong, through the C ABI (needs an MI355X): one to five K
stages (odd and even counts, ragged last stage, fewer stages than the pipeline holds),
rows and columns one 16-byte piece past and short of a 32-, 64-, 128- and 256-boundary
of the tile, and K split so that slices hold different stage counts.  int8 against the
oracle bit for bit; bf16 on integer-valued operands, whose fp32 sums are exact.
"""
import numpy as np
import pytest

from oracle import oracle
from paper_2512_13282_amd import binding as b
from paper_2512_13282_amd import inputs
import gpu_helpers as g

pytestmark = pytest.mark.gpu
I8, BF = g.I8, g.BF


@pytest.fixture(autouse=True)
def _reset_plan():
    g.unforce()
    yield
    g.unforce()


@pytest.mark.parametrize("config,bt", [(13, 0), (44, 0), (44, 1), (45, 0), (45, 1)],
                         ids=["13-row", "44-row", "44-col", "45-row", "45-col"])
@pytest.mark.parametrize("dtype", [I8, BF], ids=["i8", "bf16"])
def test_stages_and_edges(dtype, config, bt):
    piece = 16 if dtype == I8 else 8
    stage = 8 * piece
    sizes = [(256, 256), (1, piece), (32 + 1, 32 + piece), (63, 64 - piece), (129, 128 + piece), (255, 256 - piece),
             (257, 256 + piece), (400, 384)]
    depths = [stage, 2 * stage, 3 * stage, 4 * stage, 5 * stage, piece, stage + piece, 3 * stage - piece, 9 * stage + piece]
    for i, (M, N) in enumerate(sizes):
        for K in (depths if i == 0 else depths[i % 3::3]):
            if dtype == I8:
                A, B = inputs.make_inputs("int8", M, N, K, seed=700 + i)
                ref, ovf = oracle.get().gemm_i8_i32(A, B)
                assert ovf == 0
            else:
                A = inputs.small_int_bf16_matrix(M, K, seed=700 + i)
                B = inputs.small_int_bf16_matrix(K, N, seed=701 + i)
                ref = oracle.get().gemm_bf16_f64(A, B)
            for split in (1, 2, 4):
                g.force(dtype, b.GEMM_KERNEL_AUTO, config, split)
                print(f"dtype={dtype} config={config} bt={bt} {(M, N, K)} split={split}", flush=True)
                C = g.gemm_gpu_bt(dtype, A, np.ascontiguousarray(B.T)) if bt else g.gemm_gpu(dtype, A, B)
                assert np.array_equal(C.astype(np.float64), ref.astype(np.float64))
