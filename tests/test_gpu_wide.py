"""GPU parity of the sizing by repeated pairs (4- and 8-byte symbols, MIN >= 2,
chunks of at most 32 KiB): a chunk whose symbol pairs do not repeat is copied
from the input, others are staged and searched at the repeated pairs, or, when
more than 128 pairs are left, at every second position. The cases plant repeats
at and around the window's edge, at the chunk's first and last pair and across
vectors, leave 0, 1, 100, 200 and 2000 of them, use symbols that differ only in
their top byte, chunk sizes around the 16-byte vectors of 256 threads, and
launches of 1024 chunks (no scan launch) and 1025. Streams must equal the
oracle's byte for byte; nothing is written past a short capacity."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, gpu_decompress, to_device
from paper_2304_07342_amd import gpulz

pytestmark = pytest.mark.gpu


def planted(m, S, C, W, count, seed, top_only=False):
    """m distinct-looking symbols with `count` copies per chunk of 2..5 symbols
    from 1, 2, W - 1, W, W + 1 or a random distance back."""
    rng = np.random.default_rng(seed)
    t = np.uint32 if S == 4 else np.uint64
    v = rng.integers(0, 1 << (32 if S == 4 else 63), size=m, dtype=t)
    if top_only:  # 24 (56) low bits all alike
        v = (v >> t(8 * (S - 1))) << t(8 * (S - 1))
    for base in range(0, m, C):
        c = min(C, m - base)
        for k in range(count if c > 4 else 0):
            d = int(rng.choice([1, 2, W - 1, W, W + 1, int(rng.integers(1, c))]))
            L = int(rng.integers(2, 6))
            p = c - L if k % 7 == 0 else int(rng.integers(1, c))
            d = max(1, min(d, p))
            for j in range(min(L, c - p)):
                v[base + p + j] = v[base + p + j - d]
    return v.view(np.uint8)


@pytest.mark.parametrize("S", [4, 8])
@pytest.mark.parametrize("C", [1, 2, 3, 5, 255, 256, 1023, 1024, 1025, 2048, 4095, 4096, 8192])
def test_chunk_sizes(S, C):
    C = min(C, 48 * 1024 // S)  # the largest chunk there is
    for k, (W, MIN, count) in enumerate(((256, 2, 0), (32, 2, 1), (256, 2, 3), (100, 3, 20), (2, 2, 100),
                                         (256, 2, 200))):
        x = planted(2 * C + C // 3 + 1, S, C, W, min(count, C), 100 * C + k)
        x = np.concatenate([x, np.arange(k % S, dtype=np.uint8)])  # tail bytes
        print("wide", S, C, W, MIN, count, x.size, flush=True)
        want = oracle.compress(x, S, C, W, MIN)
        st, s, _, canary = gpu_compress(x, S, C, W, MIN)
        assert st == gpulz.GPULZ_OK and canary and s == want
        st, d, _, canary = gpu_decompress(s, x.size)
        assert st == gpulz.GPULZ_OK and canary and d == x.tobytes()
        st, s, n, canary = gpu_compress(x, S, C, W, MIN, capacity=len(want) - 1)
        assert st == gpulz.GPULZ_ERR_OUT_OF_SPACE and canary and n == len(want)


@pytest.mark.parametrize("S", [4, 8])
@pytest.mark.parametrize("count,top_only", [(0, False), (2, False), (2000, False), (0, True), (3, True)])
@pytest.mark.parametrize("N", [1024, 1025])
def test_many_chunks(S, count, top_only, N):
    C, W = 130, 64
    x = planted(N * C - 7, S, C, W, min(count, C), N + count, top_only)
    print("wide many", S, N, count, top_only, flush=True)
    st, s, _, canary = gpu_compress(x, S, C, W, 2)
    assert st == gpulz.GPULZ_OK and canary
    assert s == oracle.compress(x, S, C, W, 2, threads=16)


def test_dense_full_chunks():
    for S, C in ((4, 8192), (4, 4096), (8, 4096)):
        x = planted(3 * C, S, C, 256, 2000, S * C)
        print("wide dense", S, C, flush=True)
        st, s, _, canary = gpu_compress(x, S, C, 256, 2)
        assert st == gpulz.GPULZ_OK and canary and s == oracle.compress(x, S, C, 256, 2, threads=16)


def test_batch():
    import torch
    params = {4: (4096, 256, 2, 4), 8: (4096, 32, 2, 4)}
    xs, widths = [], []
    for k, (S, n, count) in enumerate([(4, 40001, 0), (8, 9000, 2), (4, 8192, 150), (8, 4097, 0), (4, 3, 0), (4, 70000, 2)]):
        C, W = params[S][:2]
        x = planted(n, S, C, W, count, 50 + k)
        xs.append(np.concatenate([x, np.arange(k % S, dtype=np.uint8)]))
        widths.append(S)
    bc = gpulz.BatchCompressor([to_device(x)[: x.size] for x in xs], widths, params)
    for _ in range(2):
        bc.run()
    torch.cuda.synchronize()
    for (st, s), x, S in zip(bc.results(), xs, widths):
        C, W, MIN, _ = params[S]
        assert st == gpulz.GPULZ_OK and s.cpu().numpy().tobytes() == oracle.compress(x, S, C, W, MIN)
