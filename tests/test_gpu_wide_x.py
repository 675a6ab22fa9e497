"""vbq_gemm_small on rows of X that lie far apart: the matrix-core kernel addresses
X with 32-bit byte offsets, so rows spanning 4 GiB or more take several launches
(and rows spanning 2 to 4 GiB one)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import matmul as omatmul  # noqa: E402
from paper_2607_02893_amd import synth  # noqa: E402
from tests import parity  # noqa: E402

pytestmark = pytest.mark.gpu

GIB = 1 << 29  # fp16 elements


@pytest.fixture(scope="module")
def vbq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2607_02893_amd import vbq as v
    return v


# rows, row stride, one width (0: mixed): one launch of a 3 GiB span; two rows and
# one; three rows at a time; 15 rows and one; single rows; M = 2 a row at a time
@pytest.mark.parametrize("y_dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("M,ldx,uniform", [(3, GIB + GIB // 2, 0), (3, 2 * GIB, 0), (8, GIB + GIB // 4, 0),
                                           (16, 4 * GIB // 15 + 7 & ~7, 0), (3, 4 * GIB, 4), (2, 4 * GIB, 2)])
def test_rows_spanning_gigabytes(vbq, M, ldx, uniform, y_dtype):
    N, K = 300, 448
    print(f"wide X: M={M} ldx={ldx} uniform={uniform} {y_dtype}", flush=True)
    bits, q, s = synth.make_matrix(synth.MatrixSpec("t", 1, 2, N, K, uniform_bits=uniform), 331)
    Wp = vbq.PackedMatrix(*vbq.pack_codes(q, s, bits))
    assert vbq.kernel_name(Wp.desc, M).startswith("vbq_mm_kernel<")
    X = synth.draw_x(synth.rng_for(337, M), M, K)
    buf = torch.empty((M - 1) * ldx + K, dtype=torch.float16, device="cuda")
    Xd = buf.as_strided((M, K), (ldx, 1))
    Xd.copy_(torch.from_numpy(X).cuda())
    Y = torch.full((M, N), 7.0, dtype=y_dtype, device="cuda")
    Wp.gemm_small(Xd, Y)
    Y = Y.cpu().numpy().astype(np.float64)
    for m in range(M):
        want = omatmul.gemv(q, s, X[m])
        bound = parity.fp32_bound(q, s, bits, X[m])
        if y_dtype == torch.float16:  # and half an ulp of fp16
            bound = bound + np.maximum(np.abs(want), 2.0 ** -14) * 2.0 ** -11 * (1 + 2.0 ** -10)
        parity.check_bound(Y[m], want, bound, what=f"row {m}")
    del buf, Xd
    torch.cuda.empty_cache()
