"""Parity and speed of the bucket encoder (1- and 2-byte symbols) off its usual
inputs. Times are compared within one process with a call that does the same work
another way, by bounds well off both sides (the figures are in the tests)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, gpu_decompress, to_device
from paper_2304_07342_amd import gpulz, synth
from test_gpu_bucket import repeats
from test_gpu_wide_routes import compress_us, device_us

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


def one_byte(kind: str, m: int, seed: int) -> np.ndarray:
    rng = np.random.default_rng(seed)
    if kind.startswith("few"):
        return rng.integers(0, int(kind[3:]), m).astype(np.uint8)
    if kind.startswith("zeros"):
        return np.where(rng.random(m) < int(kind[5:]) / 100, 0, rng.integers(1, 256, m)).astype(np.uint8)
    top = int(kind[4:])
    k = 2 * m // top + 8
    return np.resize(np.repeat(rng.integers(0, 200, k), rng.integers(1, top + 1, k)), m).astype(np.uint8)


FULL = ["few2", "few3", "few5", "zeros50", "zeros70", "zeros90", "zeros99", "runs8", "runs64", "runs600"]


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("kind", FULL)
def test_full_buckets(S, kind):
    """Tiles of few symbols, of one that holds a third, of runs of many, alone and
    in turns with text, in launches of few chunks (8-position segments up to C
    4096, 16-position ones above) and of many (16 and 32), and in a batch."""
    import torch
    t = np.uint8 if S == 1 else np.uint16
    xs = []
    for C, N in ((100, 40), (2048, 3), (4096, 2), (4097, 3), (8192, 2), (1300, 400), (4097, 300), (8192, 270)):
        m = (N - 1) * C + C // 2 + 1
        x = np.resize(one_byte(kind, min(m, 1 << 17), C), m)
        if C % 2 == 0:  # stretches of 700 in turns with text
            z = np.resize(synth.zipf_text(1 << 16, seed=C).view(np.uint8)[: 1 << 16], m)
            x = np.where(np.arange(m) // 700 % 2 == 0, x, z)
        x = x.astype(t).view(np.uint8)
        if C == 8192 and N == 2:
            xs.append(x)
        for W, MIN in ((256, 2), (128, 3)) if N < 100 else ((256, 2),):
            print("full buckets", S, kind, C, N, W, MIN, flush=True)
            want = oracle.compress(x, S, C, W, MIN, threads=16)
            st, s, _, canary = gpu_compress(x, S, C, W, MIN)
            assert st == gpulz.GPULZ_OK and canary and s == want
            st, d, _, canary = gpu_decompress(s, x.size)
            assert st == gpulz.GPULZ_OK and canary and d == x.tobytes()
    params = {S: (8192, 256, 2, 1)}
    bc = gpulz.BatchCompressor([to_device(x)[: x.size] for x in xs], [S] * len(xs), params)
    bc.run()
    torch.cuda.synchronize()
    for (st, s), x in zip(bc.results(), xs):
        assert st == gpulz.GPULZ_OK and s.cpu().numpy().tobytes() == oracle.compress(x, S, 8192, 256, 2)


@pytest.mark.parametrize("S", [1, 2, 4, 8])
def test_long_scan_chunks(S):
    """Policy 1 in chunks of more than 4096 symbols (32-position segments)."""
    C = {1: 8192, 2: 8192, 4: 5000, 8: 4097}[S]
    for kind in ("few3", "runs64", "zeros70"):
        for C1 in (4097, C):
            m = 2 * C1 + 77
            x = one_byte(kind, m, C1).astype({1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}[S]).view(np.uint8)
            for W, MIN in ((256, 2), (33, 3)):
                print("scan long", S, kind, C1, W, MIN, flush=True)
                st, s, _, canary = gpu_compress(x, S, C1, W, MIN, policy=1)
                assert st == gpulz.GPULZ_OK and canary and s == oracle.compress(x, S, C1, W, MIN, policy=1)


def test_runs_of_many_symbols_stay_in_buckets():
    """Runs of up to 64 of 200 byte values are bucketed in launches of many chunks
    (16 MiB: 9.0 times the time of Zipf bytes by the streaming parse, 5.3 by
    buckets), and launches of few chunks split the parse by 8 positions (256 KiB of
    runs of up to 8: 5.3 times by 16 positions, 3.3 by 8)."""
    zipf = synth.zipf_text(16 << 20, seed=1).view(np.uint8)
    r64 = np.resize(one_byte("runs64", 1 << 20, 1), 16 << 20)
    r8 = np.resize(one_byte("runs8", 1 << 18, 1), 1 << 18)
    us = {"zipf": compress_us(zipf, 1, 4096, 256), "runs64": compress_us(r64, 1, 4096, 256),
          "zipf few": compress_us(zipf[: 1 << 18], 1, 2048, 128), "runs8 few": compress_us(r8, 1, 2048, 128)}
    print("runs us", us, flush=True)
    assert us["runs64"] < 7.2 * us["zipf"]
    assert us["runs8 few"] < 4.3 * us["zipf few"]


@pytest.mark.parametrize("S", [1, 2, 4, 8])
@pytest.mark.parametrize("kind", ["few2", "few3", "zeros70", "zeros90", "zeros100", "runs64", "runs600"])
def test_scan_of_few_symbols(S, kind):
    """Policy 1 where many slots are equal: waves that walk slot by slot, groups of
    slots that every lane has passed, runs extended four symbols a step up to the
    chunk's end, tokens longer than the parse's segments."""
    t = {1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}[S]
    for C in (65, 1023, 1024, 2050, 4096):
        m = 2 * C + C // 3
        x = one_byte(kind, m, C).astype(t).view(np.uint8)
        for W, MIN in ((256, 2), (129, 3), (64, 2), (33, 2), (5, 2)):
            print("scan few", S, kind, C, W, MIN, flush=True)
            st, s, _, canary = gpu_compress(x, S, C, W, MIN, policy=1)
            assert st == gpulz.GPULZ_OK and canary and s == oracle.compress(x, S, C, W, MIN, policy=1)


def test_scan_time_hardly_depends_on_the_symbols():
    """Policy 1 walks slot by slot where the masks have too much to take: 4 MiB of
    bytes, W 256, nine zeros of ten, take 2.2 times the time of Zipf bytes, by masks
    4.1 times."""
    us = {}
    for kind in ("zipf", "zeros90"):
        x = synth.zipf_text(4 << 20, seed=1).view(np.uint8) if kind == "zipf" else one_byte(kind, 4 << 20, 1)
        d = to_device(x)[: x.size]
        c = gpulz.Compressor(x.size, 1, 4096, 256, 2, policy=1)
        us[kind] = device_us(lambda: c.compress_async(d))
    print("scan us", us, flush=True)
    assert us["zeros90"] < 3 * us["zipf"]
