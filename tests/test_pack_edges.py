"""The packer where its batching can go wrong: 1-bit groups are summed eight at a
time (counts that leave a remainder, alone and among other widths), units are
written by row while entries go by column, and any number of threads writes the
same bytes as one."""

import numpy as np
import pytest

from oracle import layout as olayout
from oracle import quant as oquant
from paper_2607_02893_amd import synth, vbq


@pytest.mark.parametrize("mix", [{1: 1.0}, {8: 1.0}, {1: .5, 8: .5}, {1: .3, 2: .3, 4: .4}])
@pytest.mark.parametrize("N,K,R,C", [(1, 64, 16, 1), (7, 64, 16, 1), (9, 192, 16, 2), (33, 704, 32, 3), (300, 1024, 256, 8)])
def test_pack_bytes_match_oracle_and_threads_agree(N, K, R, C, mix):
    rng = synth.rng_for(17, N, K)
    W = synth.draw_weights(rng, N, K, std=1.0) * rng.uniform(1e-4, 10, (N, 1)).astype(np.float32)
    W[0, :5] = [0.0, -0.0, 2.5, -2.5, 0.5]
    bits = synth.draw_bits(rng, N, K // 64, mix)
    q, s = oquant.quantize(W, bits)
    oblob, _ = olayout.pack(q, s, bits, R, C)
    for threads in (1, 3, 0):
        blob, _ = vbq.pack(W, bits, tile_rows=R, chunk_groups=C, n_threads=threads)
        assert np.array_equal(np.asarray(blob), oblob), threads
        blob, _ = vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C, n_threads=threads)
        assert np.array_equal(np.asarray(blob), oblob), threads


def test_queued_means_keep_their_errors():
    """A 1-bit mean beyond fp16 is refused wherever its group stands in a batch."""
    for k in (0, 7, 8, 10):
        W = np.ones((11, 64), dtype=np.float32)
        W[k] = 1e5
        with pytest.raises(vbq.VbqError) as e:
            vbq.pack(W, np.ones((11, 1), dtype=np.uint8))
        assert e.value.status == 6
