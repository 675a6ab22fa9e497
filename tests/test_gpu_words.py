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
