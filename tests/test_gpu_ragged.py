"""The matrix-core product where a unit's columns end inside a width-map word (one,
two or three of the four columns of a 16-row word, one of the two of a 32-row
word): X past the last column is never part of a sum.  X is followed by NaN in
every row, in one buffer that ends with the last row's NaN."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import matmul as omatmul  # noqa: E402
from paper_2607_02893_amd import synth  # noqa: E402
from tests import parity  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vbq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2607_02893_amd import vbq as v
    return v


@pytest.mark.parametrize("uniform", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("M", [3, 16])
@pytest.mark.parametrize("N,K,R,C", [(50, 64, 16, 1), (50, 128, 16, 2), (50, 192, 16, 3), (50, 320, 16, 5), (50, 704, 16, 6),
                                     (50, 960, 16, 15), (100, 64, 32, 1), (100, 704, 32, 3), (12400, 192, 16, 1)])
def test_columns_past_the_last_one(vbq, N, K, R, C, M, uniform):
    print(f"ragged: M={M} N={N} K={K} R={R} C={C} uniform={uniform}", flush=True)
    bits, q, s = synth.make_matrix(synth.MatrixSpec("t", N % 7, K % 5, N, K, uniform_bits=uniform), 347)
    Wp = vbq.PackedMatrix(*vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C))
    assert vbq.kernel_name(Wp.desc, M).split(",")[2].startswith("true")
    X = synth.draw_x(synth.rng_for(349, M), M, K)
    Xd = torch.full((M, K + 256), float("nan"), dtype=torch.float16, device="cuda")
    Xd[:, :K] = torch.from_numpy(X).cuda()
    Y = torch.full((M, N), 7.0, device="cuda")
    Wp.gemm_small(Xd[:, :K], Y)
    Y = Y.cpu().numpy()
    for m in range(M):
        parity.check_bound(Y[m], omatmul.gemv(q, s, X[m]), parity.fp32_bound(q, s, bits, X[m]), what=f"row {m}")
