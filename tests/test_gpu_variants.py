"""Every variant of the batch kernel for units that fill their last width-map word
(one width and mixed, four and eight waves, tiles of 16, 32 and 64 rows), the
variants for items of one word, and the sixteen-wave one-width product of one
row: the variant that the geometry is meant to reach, exact on a one-hot column,
within the bound of any float32 order of summation on random rows, and nothing
written beside the result.  Row counts leave a ragged last tile."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import matmul as omatmul  # noqa: E402
from paper_2607_02893_amd import synth  # noqa: E402
from tests import parity  # noqa: E402

pytestmark = pytest.mark.gpu

# waves, row blocks; N, K, tile rows, chunk groups
ONE_WIDTH = [(4, 1, 37, 1024, 16, 4), (8, 1, 37, 2048, 16, 8), (4, 2, 45, 128, 32, 2), (8, 2, 45, 256, 32, 2)]
CASES = ([(f"vbq_mm_kernel<{nw},{rb},false,{c}>", M, N, K, R, C, 1 << c)
          for nw, rb, N, K, R, C in ONE_WIDTH for c in range(4) for M in (2, 3, 16)]
         + [("vbq_mm_kernel<8,2,false>", M, 45, 256, 32, 2, 0) for M in (3, 16)]
         + [("vbq_mm_kernel<4,1,false,-2>", M, 12310, 256, 16, 4, 0) for M in (3, 16)]
         + [("vbq_mm_kernel<8,4,false,-2>", M, 300, 320, 64, 1, 0) for M in (3, 16)]
         + [(f"vbq_mv_kernel<1,16,{c}>", 1, 37, 576, 16, 1, 1 << c) for c in range(4)])


@pytest.fixture(scope="module")
def vbq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2607_02893_amd import vbq as v
    return v


@pytest.mark.parametrize("name,M,N,K,R,C,uniform", CASES)
def test_variant(vbq, name, M, N, K, R, C, uniform):
    print(f"{name} M={M} N={N} K={K} R={R} C={C} uniform={uniform}", flush=True)
    bits, q, s = synth.make_matrix(synth.MatrixSpec("t", N % 11, K % 7, N, K, uniform_bits=uniform), 359)
    Wp = vbq.PackedMatrix(*vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C))
    assert vbq.kernel_name(Wp.desc, M) == name
    X = synth.draw_x(synth.rng_for(367, M), M, K)
    if M > 1:
        X[0] = 0
        X[0, K - 1] = 1.0
    Xd = torch.full((M, K + 8), float("nan"), dtype=torch.float16, device="cuda")
    Xd[:, :K] = torch.from_numpy(X).cuda()
    Yd = torch.full((M, N + 3), 7.0, device="cuda")
    Wp.gemm_small(Xd[:, :K], Yd[:, :N])
    Y = Yd.cpu().numpy()
    assert np.all(Y[:, N:] == 7.0)
    if M > 1:
        assert np.array_equal(Y[0, :N].astype(np.float64), omatmul.gemv(q, s, X[0]))
    for m in range(M):
        parity.check_bound(Y[m, :N], omatmul.gemv(q, s, X[m]), parity.fp32_bound(q, s, bits, X[m]), what=f"row {m}")
