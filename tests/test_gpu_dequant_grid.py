"""vbq_dequant's split of the tiles over workgroups: unit counts that do not fill the
last workgroup, units cut into slices of several words, one word and less, and
grids large enough for whole units; and the variant for one-column units of 16
rows, with a last tile of fewer rows."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import matmul as omatmul  # noqa: E402
from paper_2607_02893_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vbq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2607_02893_amd import vbq as v
    return v


# N, K, tile rows, chunk groups: three units; five, and seven of one column; one
# unit of 128 words; two of 32 words; 1200 tiles of five (whole units); 4100 tiles of
# one; one column of 1, 5 and 14 rows in the last tile; one-column units of 32 rows
@pytest.mark.parametrize("N,K,R,C", [(100, 576, 0, 0), (70, 1280, 64, 4), (40, 448, 16, 1), (300, 2048, 256, 32),
                                     (30, 16384, 16, 128), (19200, 320, 16, 1), (65590, 64, 16, 1),
                                     (17, 256, 0, 0), (5, 64, 0, 0), (30, 128, 0, 0), (45, 192, 32, 1)])
def test_dequant_over_the_grid(vbq, N, K, R, C):
    print(f"dequant grid N={N} K={K} R={R} C={C}", flush=True)
    bits, q, s = synth.make_matrix(synth.MatrixSpec("t", N % 11, K % 7, N, K), 353)
    Wp = vbq.PackedMatrix(*vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C))
    want = torch.from_numpy(omatmul.dequant(q, s).astype(np.float32))
    buf = torch.full((N * K + 64,), 7.0, device="cuda")
    out = Wp.dequant(buf[:N * K].view(N, K))
    assert torch.equal(out.cpu(), want)
    assert torch.all(buf[N * K:] == 7.0)
