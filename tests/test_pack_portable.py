"""The packer's two quantizers give the same bytes: vbq_pack.cpp built without its
AVX2 code against the library (which uses it where the processor has it) and
the oracle, with ties, both zeros, zero and smallest scales, and every refusal."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import layout as olayout
from oracle import quant as oquant
from paper_2607_02893_amd import build, synth, vbq


@pytest.fixture(scope="module")
def portable(tmp_path_factory):
    clang = os.path.join(build.ROCM, "llvm", "bin", "clang++")
    clang = clang if os.path.exists(clang) else shutil.which("amdclang++")
    if not clang:
        pytest.skip("no clang++ (the packer needs _Float16)")
    so = str(tmp_path_factory.mktemp("portable") / "libvbq_pack_portable.so")
    subprocess.run([clang, "-O3", "-std=c++17", "-fPIC", "-shared", "-DVBQ_PACK_PORTABLE",
                    os.path.join(build.CSRC, "vbq_pack.cpp"), "-o", so, "-lpthread"], check=True)
    lib = ctypes.CDLL(so)
    for name in ("vbq_pack_size", "vbq_pack", "vbq_pack_codes", "vbq_status_string"):
        getattr(lib, name).argtypes = getattr(vbq.lib(), name).argtypes
        getattr(lib, name).restype = getattr(vbq.lib(), name).restype
    return lib


def _both(portable, monkeypatch, call):
    """call() with the library and with the portable build: bytes, or the error's status."""
    out = []
    for lib in (vbq.lib(), portable):
        with monkeypatch.context() as m:
            m.setattr(vbq, "_lib", lib)
            try:
                out.append(np.asarray(call()[0]).copy())
            except vbq.VbqError as e:
                out.append(e.status)
    return out


def _weights(rng, N, K):
    """Rows of very different magnitude; group j % 8 == 0 .. 4 of each row: ties at
    every width, both zeros, all zeros, subnormal scales, one large weight."""
    W = synth.draw_weights(rng, N, K, std=1.0) * rng.uniform(1e-4, 10, (N, 1)).astype(np.float32)
    g = W.reshape(N, K // 64, 64)
    ties = ((np.arange(64) % 15 - 7) / 2).astype(np.float32)
    g[:, 0::8] = ties / 8
    g[:, 0::8, 0] = 127 / 8
    g[:, 1::8, ::2] = 0.0
    g[:, 1::8, 1::4] = -0.0
    g[:, 2::8] = 0.0
    g[:, 3::8] *= 1e-7
    g[:, 4::8, 63] = -60000.0
    return W


@pytest.mark.parametrize("mix", [{1: 1.0}, {2: 1.0}, {4: 1.0}, {8: 1.0}, {1: .5, 2: .2, 4: .2, 8: .1}])
@pytest.mark.parametrize("N,K,R,C", [(7, 64, 16, 1), (33, 704, 32, 3), (300, 1024, 256, 8)])
def test_both_quantizers_give_the_same_bytes(portable, monkeypatch, N, K, R, C, mix):
    rng = synth.rng_for(19, N, K)
    W = _weights(rng, N, K)
    bits = synth.draw_bits(rng, N, K // 64, mix)
    q, s = oquant.quantize(W, bits)
    want, _ = olayout.pack(q, s, bits, R, C)
    for got in _both(portable, monkeypatch, lambda: vbq.pack(W, bits, tile_rows=R, chunk_groups=C)):
        assert np.array_equal(got, want)
    for got in _both(portable, monkeypatch, lambda: vbq.pack_codes(q, s, bits, tile_rows=R, chunk_groups=C)):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("b", [1, 2, 4, 8])
@pytest.mark.parametrize("bad,status", [(np.nan, 5), (-np.nan, 5), (np.inf, 5), (-np.inf, 5), (1e8, 6), (-1e8, 6)])
@pytest.mark.parametrize("at", [0, 17, 63])
def test_both_quantizers_refuse_the_same(portable, monkeypatch, b, bad, status, at):
    W = np.ones((11, 128), dtype=np.float32)
    W[9, 64 + at] = bad
    bits = np.full((11, 2), b, dtype=np.uint8)
    assert _both(portable, monkeypatch, lambda: vbq.pack(W, bits)) == [status, status]
