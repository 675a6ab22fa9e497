"""The register lookup of entries from width-map words (word_entries), at the
sizes where it can go wrong: units of more than 64 words (a second scan), units
of less than one word, last words that are partly padding, ragged tiles of
every tile height, one width alone, and an output that is only 4-byte aligned."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import matmul as omatmul  # noqa: E402
from paper_2607_02893_amd import synth  # noqa: E402
from tests import parity  # noqa: E402

pytestmark = pytest.mark.gpu

# N, K, tile rows, chunk groups
GEOMS = [(700, 2112, 256, 32), (515, 4160, 128, 64), (65, 4096, 64, 64), (31, 8256, 16, 128), (33, 448, 32, 7),
         (17, 64, 16, 1), (1, 192, 256, 2)]


@pytest.fixture(scope="module")
def vbq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2607_02893_amd import vbq as v
    return v


def _packed(vbq, N, K, R, C, uniform=0):
    bits, q, s = synth.make_matrix(synth.MatrixSpec("t", N % 11, K % 7, N, K, uniform_bits=uniform), 307)
    blob, d = vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C)
    return vbq.PackedMatrix(blob, d), bits, q, s


@pytest.mark.parametrize("uniform", [0, 1, 8])
@pytest.mark.parametrize("N,K,R,C", GEOMS)
def test_dequant_exact_and_unaligned(vbq, N, K, R, C, uniform):
    print(f"dequant N={N} K={K} R={R} C={C} uniform={uniform}", flush=True)
    Wp, _, q, s = _packed(vbq, N, K, R, C, uniform)
    want = torch.from_numpy(omatmul.dequant(q, s).astype(np.float32))
    buf = torch.full((N * K + 3,), 7.0, device="cuda")
    out = buf[1:1 + N * K]  # 4-byte aligned only
    st = vbq.lib().vbq_dequant(ctypes.byref(Wp.desc), ctypes.c_void_p(Wp.blob.data_ptr()), ctypes.c_void_p(out.data_ptr()),
                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    assert torch.equal(out.cpu().view(N, K), want)
    assert buf[0].item() == 7.0 and torch.all(buf[1 + N * K:] == 7.0)  # nothing written outside


# the matrix-core product: also a grid beyond the wave-pair kernel's (two rows),
# and the variant for items of one word (16-row tiles beyond 768 of them, 64-row tiles)
MM_GEOMS = GEOMS[:6] + [(33000, 256, 16, 1), (33000, 256, 64, 1)]


@pytest.mark.parametrize("uniform", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("M", [2, 5, 16])
@pytest.mark.parametrize("N,K,R,C", MM_GEOMS)
def test_batch_products_within_the_float32_bound(vbq, N, K, R, C, M, uniform):
    """Row 0 of X is a one-hot column (exact: a level times its scale), the others
    random, within the bound of any float32 order of summation; padded X and Y."""
    print(f"gemm M={M} N={N} K={K} R={R} C={C} uniform={uniform}", flush=True)
    Wp, bits, q, s = _packed(vbq, N, K, R, C, uniform)
    if M > 2 or uniform or Wp.desc.n_units > 2048:
        assert vbq.kernel_name(Wp.desc, M).startswith("vbq_mm_kernel<")
    if N == 33000 and not uniform:
        assert vbq.kernel_name(Wp.desc, M).endswith(",-2>") or (M == 2 and Wp.desc.n_units <= 2048)
    X = synth.draw_x(synth.rng_for(311, M), M, K)
    X[0] = 0
    X[0, K - 1] = 1.0
    Xd = torch.zeros((M, K + 8), dtype=torch.float16, device="cuda")
    Xd[:, :K] = torch.from_numpy(X).cuda()
    Yd = torch.full((M, N + 3), 7.0, device="cuda")
    Wp.gemm_small(Xd[:, :K], Yd[:, :N])
    Y = Yd.cpu().numpy()
    assert np.all(Y[:, N:] == 7.0)
    assert np.array_equal(Y[0, :N].astype(np.float64), omatmul.gemv(q, s, X[0]))
    for m in (1, M - 1):
        parity.check_bound(Y[m, :N], omatmul.gemv(q, s, X[m]), parity.fp32_bound(q, s, bits, X[m]), what=f"row {m}")
