"""GPU parity of the bucket encoder (1- and 2-byte symbols, MIN >= 2): it
searches a chunk in tiles of 1024 positions through 2-symbol buckets, tells
matches of up to 5 symbols from the bucket entries, extends longer ones in the
parse and compares 2-byte symbols through their low bytes. The cases sit where
that can go wrong: chunk sizes around the tile and segment edges, one symbol,
the largest chunk; windows around a bucket block; matches of 5 to 7 symbols
and of the whole window, one or several candidates; symbols that differ only
in their high byte; matches cut by the chunk end; buckets too full for it
(long runs). Streams must equal the oracle's byte for byte, in launches of few
chunks (16 waves each) and of many (4 waves each)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, gpu_decompress
from paper_2304_07342_amd import gpulz, synth

pytestmark = pytest.mark.gpu


def repeats(m: int, S: int, seed: int, span: int) -> np.ndarray:
    """m symbols out of `span` values (2-byte symbols: half of them 256 above
    the others, so that low bytes collide) with copies of 2..9, 30 and 300
    symbols from 1..300 back, some copied twice."""
    rng = np.random.default_rng(seed)
    v = rng.integers(0, span, size=m)
    if S == 2:
        v = v + 256 * rng.integers(0, 2, size=m) * (seed % 2)
    v = v.astype(np.uint8 if S == 1 else np.uint16)
    p = 2
    while p < m:
        L = int(rng.choice([2, 3, 5, 6, 7, 8, 9, 30, 300], p=[.2, .15, .15, .15, .1, .1, .05, .08, .02]))
        for _ in range(int(rng.integers(1, 3))):
            d = int(rng.integers(1, min(p, 300) + 1))
            L = min(L, m - p)
            for k in range(L):
                v[p + k] = v[p + k - d]
            p += L
            if p >= m:
                break
        p += int(rng.integers(0, 12))
    return v.view(np.uint8)


SIZES = [1, 2, 15, 63, 1023, 1024, 1025, 1026, 1300, 2047, 2050, 4097, 8191, 8192]


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("C", SIZES)
def test_chunk_sizes(S, C):
    for k, W in enumerate((1, 2, 127, 128, 129, 256)):
        for MIN in (2, 3, 6, 7) if C <= 4096 else (2,):
            x = repeats(2 * C + C // 3, S, 31 * C + 8 * k + MIN, 9 if k % 2 else 60)
            print("bucket", S, C, W, MIN, x.size, flush=True)
            st, s, _, canary = gpu_compress(x, S, C, W, MIN)
            assert st == gpulz.GPULZ_OK and canary
            assert s == oracle.compress(x, S, C, W, MIN)
            st, d, _, canary = gpu_decompress(s, x.size)
            assert st == gpulz.GPULZ_OK and canary and d == x.tobytes()


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("kind", ["repeats", "wide", "runs", "few", "uniform"])
def test_many_chunks(S, kind):
    C, n = 1300, 600 * 1300 + 77
    if kind == "repeats":
        x = repeats(n, S, 5, 40)
    elif kind == "wide":  # every chunk's symbols span the whole range
        x = np.tile(repeats(1 << 16, S, 7, 60), -(-n * S >> 16))[: n * S].copy()
        x[:: 997] ^= 0x80
    elif kind == "runs":
        x = np.tile(synth.runs(1 << 16, S, 3), -(-n // (1 << 16)))[: n * S]
    elif kind == "few":
        x = synth.small_alphabet(n, S, 4, alphabet=3)
    else:
        x = synth.uniform_bytes(n * S, 6)
    for W, MIN in ((256, 2), (100, 3)):
        print("bucket many", S, kind, W, MIN, flush=True)
        st, s, _, canary = gpu_compress(x, S, C, W, MIN)
        assert st == gpulz.GPULZ_OK and canary
        assert s == oracle.compress(x, S, C, W, MIN, threads=16)
