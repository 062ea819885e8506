"""GPU parity of the wave decoder (1- and 2-byte symbols, streams and batches
of more than 1536 chunks): one wavefront per chunk, 64 tokens a round, a ring
of 1024 symbols, steps of at most 512 + 255 symbols, 256 symbols written out
at once. The streams have chunks below and above each of these, outputs that
are not 16-byte aligned, pointers of 255 symbols (a round of them takes several
steps), chains of short offsets within 64 symbols and offset 256; every
mutated stream's verdict must equal the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_decompress, to_device
from paper_2304_07342_amd import gpulz, synth
from test_gpu_bucket import repeats

pytestmark = pytest.mark.gpu

N = 1600


def _content(kind, m, S, seed):
    if kind == "repeats":
        return np.tile(repeats(1 << 15, S, seed, 30), -(-m * S // (S << 15)))[: m * S]
    if kind == "runs":
        return np.tile(synth.runs(1 << 15, S, seed), -(-m * S // (S << 15)))[: m * S]
    return synth.uniform_bytes(m * S, seed)


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("C", [1, 7, 64, 255, 300, 768, 1024, 1030, 2500, 4097])
def test_round_trip(S, C):
    for kind in ("repeats", "runs", "uniform"):
        for W, MIN in ((256, 2), (5, 1)):
            x = _content(kind, N * C + C // 2, S, 3 + C)
            print("wave decode", S, C, kind, W, MIN, flush=True)
            s = oracle.compress(x, S, C, W, MIN, threads=16)
            st, d, n, canary = gpu_decompress(s, x.size)
            assert st == gpulz.GPULZ_OK and canary and n == x.size
            assert d == x.tobytes()


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("kind", ["repeats", "runs"])
def test_mutations(S, kind):
    C = 70
    x = _content(kind, N * C, S, 11)
    s = np.frombuffer(oracle.compress(x, S, C, 256, 2, threads=16), dtype=np.uint8)
    rng = np.random.default_rng(5)
    chunks = N
    table = s[64:64 + 8 * chunks].view(np.uint32).reshape(-1, 2).astype(np.int64)
    starts = 64 + 8 * chunks + np.concatenate([[0], np.cumsum(table.sum(1))])
    for k in range(60):
        t = s.copy()
        i = int(rng.integers(chunks))
        F, P = int(table[i, 0]), int(table[i, 1])
        what = k % 4
        if what == 0:  # a flag bit
            t[starts[i] + int(rng.integers(F))] ^= 1 << int(rng.integers(8))
        elif what == 1:  # a payload byte
            t[starts[i] + F + int(rng.integers(P))] = int(rng.integers(256))
        elif what == 2:  # one byte more or less of flags, the record's size kept
            e = t[64 + 8 * i: 72 + 8 * i].view(np.uint32)
            d = 1 if rng.integers(2) else -1
            e[0], e[1] = F + d, P - d
        else:  # the last chunk's last payload byte
            t[-1] ^= 1 + int(rng.integers(255))
        want, data, _ = oracle.decompress_status(t.tobytes())
        print("wave decode mutation", S, kind, k, what, i, "oracle", want, flush=True)
        st, d, _, canary = gpu_decompress(t.tobytes(), x.size)
        assert canary and (st == gpulz.GPULZ_OK) == (want == 0)
        if want == 0:
            assert d == data


def test_batch():
    import torch
    srcs, want = [], []
    for k, (S, C, n) in enumerate([(1, 64, 64 * 900 + 5), (2, 50, 100 * 700), (4, 128, 512 * 40), (1, 3000, 40000),
                                   (8, 64, 512 * 9 + 3), (2, 1024, 2048 * 33 + 1)]):
        x = _content("repeats" if S <= 2 else "uniform", n // S + 1, S, 20 + k)[:n]
        want.append(x.tobytes())
        srcs.append(to_device(np.frombuffer(oracle.compress(x, S, C, 256, 2, threads=16), dtype=np.uint8)))
    bd = gpulz.BatchDecompressor(srcs, [len(w) for w in want])
    bd.run()
    torch.cuda.synchronize()
    for (st, y), w in zip(bd.results(), want):
        assert st == gpulz.GPULZ_OK and y.cpu().numpy().tobytes() == w
