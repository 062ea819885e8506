"""Speed and parity of 4- and 8-byte symbols off the noisy-field path. Times are
compared within one process with a call that does the same work another way, by
bounds well off both sides (the figures are in the tests)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, to_device
from paper_2304_07342_amd import gpulz, synth

pytestmark = pytest.mark.gpu


def device_us(run):
    import torch
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(12):
        e[0].record()
        for _ in range(4):
            run()
        e[1].record()
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) / 4 * 1e3)
    return best


def compress_us(x, S, C, W, MIN=2):
    d = to_device(x)[: x.size]
    c = gpulz.Compressor(x.size, S, C, W, MIN)
    return device_us(lambda: c.compress_async(d))


def test_records_of_256_chunks():
    """256 chunks of noise are written about as fast as 64 of them (13.0 and 12.0
    us); with the record sizes chosen by address, which made every workgroup read
    its launch packet, they took 25.5 and 15.1."""
    x = synth.uniform_bytes(4 << 20, 1)
    us = {n: compress_us(x[: n * 16384], 4, 4096, 256) for n in (64, 256)}
    print("wide records us", us, flush=True)
    assert us[256] < 1.35 * us[64]


def repetitive(kind: str, m: int, S: int, seed: int) -> np.ndarray:
    rng = np.random.default_rng(seed)
    t = {4: np.uint32, 8: np.uint64}[S]
    if kind == "few":
        v = rng.integers(0, 16, m)
    elif kind == "zeros":
        v = np.zeros(m)
    elif kind == "nearly zeros":  # fewer than one turn in 128
        v = np.where(rng.random(m) < 1 / 400, rng.integers(1, 9, m), 0)
    elif kind == "half zeros":
        v = np.where(np.arange(m) // 97 % 2 == 1, 0, rng.integers(0, 1 << 31, m))
    else:  # runs of 1..64 symbols
        v = np.repeat(rng.integers(0, 200, m // 16 + 2), rng.integers(1, 65, m // 16 + 2))[:m]
        v = np.resize(v, m)
    return v.astype(t).view(np.uint8)


KINDS = ["few", "zeros", "nearly zeros", "half zeros", "runs"]


@pytest.mark.parametrize("S", [4, 8])
@pytest.mark.parametrize("kind", KINDS)
def test_repetitive_chunks(S, kind):
    """Launches of up to 512 chunks size repetitive chunks with 16 waves, those
    of nearly one run with one; longer chunks (C above 4096) with one."""
    for C, N in ((1, 3), (2, 5), (60, 513), (60, 512), (300, 40), (1025, 9), (4095, 3), (4096, 2), (8192 // (S // 4), 2),
                 (1000, 600)):
        x = repetitive(kind, (N - 1) * C + C // 2 + 1, S, C + N)
        x = np.concatenate([x, np.arange(C % S, dtype=np.uint8)])
        for W, MIN in ((256, 2), (128, 2), (31, 3)):
            print("wide repetitive", S, kind, C, N, W, MIN, flush=True)
            want = oracle.compress(x, S, C, W, MIN, threads=16)
            st, s, _, canary = gpu_compress(x, S, C, W, MIN)
            assert st == gpulz.GPULZ_OK and canary and s == want
            st, s, n, canary = gpu_compress(x, S, C, W, MIN, capacity=len(want) - 1)
            assert st == gpulz.GPULZ_ERR_OUT_OF_SPACE and canary and n == len(want)


def test_repetitive_batch():
    import torch
    params = {4: (4096, 256, 2, 4), 8: (2048, 64, 2, 4)}
    xs, widths = [], []
    for k, kind in enumerate(KINDS * 2):
        S = 4 if k < 5 else 8
        xs.append(repetitive(kind, 9000 + 1111 * k, S, k))
        widths.append(S)
    bc = gpulz.BatchCompressor([to_device(x)[: x.size] for x in xs], widths, params)
    for _ in range(2):
        bc.run()
    torch.cuda.synchronize()
    print("wide repetitive batch", flush=True)
    for (st, s), x, S in zip(bc.results(), xs, widths):
        assert st == gpulz.GPULZ_OK and s.cpu().numpy().tobytes() == oracle.compress(x, S, *params[S][:3])


@pytest.mark.parametrize("S,C", [(4, 4096), (8, 2048)])
def test_repetitive_chunks_are_split(S, C):
    """64 chunks out of 16 values: about the time of the split parse that takes
    MIN = 1 (S = 4: 218 us); one wave a chunk took 6.8 times that (S = 8: 122
    us, 6.7 times)."""
    x = repetitive("few", 64 * C, S, 1)
    us = {MIN: compress_us(x, S, C, 256, MIN) for MIN in (1, 2)}
    print("wide repetitive us", S, us, flush=True)
    assert us[2] < 2.5 * us[1]
