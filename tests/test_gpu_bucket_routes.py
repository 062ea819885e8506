"""Parity and speed of the bucket encoder (1- and 2-byte symbols) off its usual
inputs. Times are compared within one process with a call that does the same work
another way, by bounds well off both sides (the figures are in the tests)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, gpu_decompress, to_device
from paper_2304_07342_amd import gpulz, synth
from test_gpu_bucket import repeats
from test_gpu_wide_routes import compress_us

pytestmark = pytest.mark.gpu


def two_bytes(kind: str, m: int, seed: int) -> np.ndarray:
    """uint16 symbols that span 256 values or more."""
    rng = np.random.default_rng(seed)
    codes = synth.laplace_codes(m, seed=seed)
    if kind == "swapped":
        v = codes.byteswap()
    elif kind == "scaled":
        v = rng.integers(0, 256, m) << 8
    elif kind == "scaled text":
        v = synth.zipf_text(m, seed=seed).view(np.uint8)[:m].astype(np.uint16) << 8
    elif kind == "both bytes alike":
        v = rng.integers(0, 256, m) * 257
    elif kind == "repeats":
        v = repeats(m, 1, seed, 30)[:m].astype(np.uint32) * 0x3C5
    else:  # constant but for single symbols far away
        v = np.where(rng.random(m) < 1 / 300, rng.integers(0, 1 << 16, m), 77)
    return v.astype(np.uint16).view(np.uint8)


@pytest.mark.parametrize("kind", ["swapped", "scaled", "scaled text", "both bytes alike", "repeats", "constant"])
def test_wide_ranges(kind):
    for C, N in ((1, 5), (5, 40), (1023, 9), (2048, 300), (4096, 3), (8192, 2), (700, 1100)):
        x = two_bytes(kind, (N - 1) * C + C // 2 + 1, C)
        for W, MIN in ((256, 2), (100, 3), (31, 2)):
            print("two bytes", kind, C, N, W, MIN, flush=True)
            st, s, _, canary = gpu_compress(x, 2, C, W, MIN)
            assert st == gpulz.GPULZ_OK and canary and s == oracle.compress(x, 2, C, W, MIN, threads=16)


def test_scaled_symbols_are_told_apart():
    """8-bit noise scaled by 256 takes the time of the noise itself (16 MiB, C
    2048, W 128: 113 and 117 us); by the low byte, alike in all, it took 1358."""
    v = synth.uniform_bytes(8 << 20, 3)
    us = {k: compress_us((v.astype(np.uint16) << k).view(np.uint8), 2, 2048, 128) for k in (0, 8)}
    print("scaled us", us, flush=True)
    assert us[8] < 2.5 * us[0]
