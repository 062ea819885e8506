"""GPU decoding of 1- and 2-byte chunks without a pointer and of chunks that are
too long for the workgroup decoder, in streams of few chunks (one workgroup
each) and of many (one wave each). Bytes and verdicts must equal the oracle's; a
set flag in a record that is as long as its literals is a corrupt one. Decoding
random uint16 symbols must stay a copy: the same bytes as uint32 symbols take the
workgroup's copy, and token by token they took 3.4 times as long, so the bound of
twice that time lies well off both."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_decompress, to_device
from paper_2304_07342_amd import gpulz, synth
from test_gpu_bucket import repeats

pytestmark = pytest.mark.gpu


def half_literal(m: int, S: int, C: int, seed: int) -> np.ndarray:
    """Every second chunk random, the others with runs."""
    x = synth.uniform_bytes(m * S, seed).reshape(-1)
    r = np.tile(synth.runs(1 << 14, S, seed), -(-m >> 14))[: m * S]
    odd = (np.arange(m * S) // (C * S)) % 2 == 1
    return np.where(odd, r, x).astype(np.uint8)


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("C,N", [(1, 3000), (5, 2000), (64, 5000), (250, 1500), (1000, 2100), (1021, 1900)])
def test_literal_chunks_round_trip(S, C, N):
    for kind in ("uniform", "half"):
        m = N * C - C // 2
        x = synth.uniform_bytes(m * S, 7) if kind == "uniform" else half_literal(m, S, C, 7)
        for W in (1, 200):
            print("literal decode", S, C, N, kind, W, flush=True)
            s = oracle.compress(x, S, C, W, 3 if S == 1 else 2, threads=16)
            st, d, n, canary = gpu_decompress(s, x.size)
            assert st == gpulz.GPULZ_OK and canary and n == x.size and d == x.tobytes()


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("N", [40, 3000])
def test_flag_set_in_a_literal_record(S, N):
    C = 100
    x = synth.uniform_bytes(N * C * S, 3)
    s = np.frombuffer(oracle.compress(x, S, C, 1, 2, threads=16), dtype=np.uint8)
    table = s[64:64 + 8 * N].view(np.uint32).reshape(-1, 2).astype(np.int64)
    starts = 64 + 8 * N + np.concatenate([[0], np.cumsum(table.sum(1))])
    rng = np.random.default_rng(2)
    for k in range(12):
        i = int(rng.integers(N))
        assert table[i, 0] == 13 and table[i, 1] == C * S
        t = s.copy()
        t[starts[i] + (0, 12, int(rng.integers(13)))[k % 3]] ^= 1 << int(rng.integers(8))
        want, _, _ = oracle.decompress_status(t.tobytes())
        print("literal flag", S, N, k, i, "oracle", want, flush=True)
        st, _, _, canary = gpu_decompress(t.tobytes(), x.size)
        assert canary and want != 0 and st != gpulz.GPULZ_OK


LONG = [(1, 4097), (1, 20000), (2, 5000), (2, 20000), (4, 4097), (4, 12000), (8, 2049), (8, 6000)]


def _long_content(kind, m, S, seed):
    if kind == "uniform":
        return synth.uniform_bytes(m * S, seed)
    if kind == "runs":
        return synth.runs(m, S, seed)
    if kind == "few":
        return synth.small_alphabet(m, S, seed, alphabet=5)
    x = synth.mixed(m * S, S, seed)
    return x[: m * S]


@pytest.mark.parametrize("S,C", LONG)
@pytest.mark.parametrize("kind", ["uniform", "runs", "few", "mixed"])
def test_long_chunks(S, C, kind):
    m = 3 * C + C // 3
    x = np.concatenate([_long_content(kind, m, S, C), np.arange(S - 1, dtype=np.uint8)])
    for W, MIN in ((256, 2), (7, 1)):
        s = oracle.compress(x, S, C, W, MIN)
        print("long decode", S, C, kind, W, MIN, flush=True)
        st, d, n, canary = gpu_decompress(s, x.size)
        assert st == gpulz.GPULZ_OK and canary and n == x.size and d == x.tobytes()


@pytest.mark.parametrize("S,C", LONG)
def test_long_chunk_mutations(S, C):
    m = 2 * C
    x = np.concatenate([_long_content("mixed", C, S, 1), _long_content("few", C, S, 2)])
    s = np.frombuffer(oracle.compress(x, S, C, 256, 2), dtype=np.uint8)
    table = s[64:80].view(np.uint32).reshape(-1, 2).astype(np.int64)
    starts = 80 + np.concatenate([[0], np.cumsum(table.sum(1))])
    rng = np.random.default_rng(S * C)
    for k in range(24):
        t = s.copy()
        i = k % 2
        F, P = int(table[i, 0]), int(table[i, 1])
        if k % 3 == 0:
            t[starts[i] + int(rng.integers(F))] ^= 1 << int(rng.integers(8))
        elif k % 3 == 1:
            t[starts[i] + F + int(rng.integers(P))] = int(rng.integers(256))
        else:
            e = t[64 + 8 * i: 72 + 8 * i].view(np.uint32)
            d = 1 if rng.integers(2) else -1
            e[0], e[1] = F + d, P - d
        want, data, _ = oracle.decompress_status(t.tobytes())
        print("long decode mutation", S, C, k, "oracle", want, flush=True)
        st, d, _, canary = gpu_decompress(t.tobytes(), x.size)
        assert canary and (st == gpulz.GPULZ_OK) == (want == 0)
        if want == 0:
            assert d == data


def _decode_us(stream, n):
    import torch
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = torch.empty(gpulz.gpulz_decompress_workspace_size(stream.numel()), dtype=torch.uint8, device="cuda")
    meta = torch.zeros(2, dtype=torch.int64, device="cuda")
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(12):
        e[0].record()
        for _ in range(4):
            assert gpulz.gpulz_decompress(stream.data_ptr(), stream.numel(), out.data_ptr(), n, meta.data_ptr(),
                                          meta.data_ptr() + 8, ws.data_ptr(), ws.numel(),
                                          torch.cuda.current_stream().cuda_stream) == 0
        e[1].record()
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) / 4 * 1e3)
    return best


def test_random_symbols_are_copied():
    n = 32 << 20
    x = to_device(synth.uniform_bytes(n, 5))
    us = {S: _decode_us(gpulz.compress(x, S, 4096 // S * 2, 64, 2), n) for S in (2, 4)}
    print("random decode us", us, flush=True)
    assert us[2] < 2 * us[4]


def _batch_us(bd):
    import torch
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(12):
        e[0].record()
        for _ in range(4):
            bd.run()
        e[1].record()
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) / 4 * 1e3)
    return best


def test_few_narrow_chunks_in_a_wide_batch():
    """Which decoder the narrow chunks of a batch take goes by their own number:
    counted with the wide ones, a hundred of them once went to waves, one chunk
    each, after the wide chunks: 102 us where the two batches apart take 88.
    Decoded beside the wide ones they take 69 together."""
    wide = synth.uniform_bytes(4 << 20, 3)
    narrow = synth.zipf_text(100_000, seed=4).view(np.uint8)
    us = {}
    for name, items in (("wide", [(wide, 4)] * 16), ("narrow", [(narrow, 1)] * 4),
                        ("both", [(wide, 4)] * 16 + [(narrow, 1)] * 4)):
        made = gpulz.BatchCompressor([to_device(x) for x, _ in items], [S for _, S in items])
        made.run()
        bd = gpulz.BatchDecompressor([s.clone() for _, s in made.results()], [x.size for x, _ in items])
        us[name] = _batch_us(bd)
        for (st, y), (x, _) in zip(bd.results(), items):
            assert st == gpulz.GPULZ_OK and y.cpu().numpy().tobytes() == x.tobytes()
    print("batch decode us", us, flush=True)
    assert us["both"] < us["wide"] + us["narrow"]


@pytest.mark.parametrize("q", [1, 30])
def test_batch_with_every_route(q):
    """Narrow buffers of few and of many chunks, literal, long and wide ones."""
    rng = np.random.default_rng(q)
    srcs, want = [], []
    for S, C, n in ((1, 64, 4000), (2, 100, 3001), (1, 9000, 30000), (2, 2048, 9000), (4, 4096, 20000), (8, 5000, 50000)):
        for k in range(q):
            x = repeats(n // S + 1, S, 5 + k, 30)[:n] if S <= 2 and k % 2 else synth.uniform_bytes(n, k)
            want.append(x.tobytes())
            srcs.append(to_device(np.frombuffer(oracle.compress(x, S, C, 256, 2), dtype=np.uint8)))
    order = rng.permutation(len(srcs))
    bd = gpulz.BatchDecompressor([srcs[k] for k in order], [len(want[k]) for k in order])
    print("batch routes", q, flush=True)
    bd.run()
    for (st, y), k in zip(bd.results(), order):
        assert st == gpulz.GPULZ_OK and y.cpu().numpy().tobytes() == want[k]


def _kernels(run):
    """Kernels that a call launches: the nodes of its captured graph."""
    import ctypes
    import torch
    run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        run()
    hip = ctypes.CDLL("libamdhip64.so")
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("kind,S,nbytes,most", [("codes", 2, 64 << 10, 2), ("field", 4, 40_000, 2), ("codes", 2, 8 << 20, 3)])
def test_launches(kind, S, nbytes, most):
    """A stream (or the streams of a batch) below 64 KiB is decoded without a
    launch of the wave decoder, which would leave at once."""
    import torch
    x = synth.laplace_codes(nbytes // 2, seed=1).view(np.uint8) if S == 2 else synth.uniform_bytes(nbytes, 1)
    s = gpulz.compress(to_device(x), S, 2048, 128, 2).clone()
    out = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ws = torch.empty(gpulz.gpulz_decompress_workspace_size(s.numel()), dtype=torch.uint8, device="cuda")
    meta = torch.zeros(2, dtype=torch.int64, device="cuda")

    def run():
        assert gpulz.gpulz_decompress(s.data_ptr(), s.numel(), out.data_ptr(), nbytes, meta.data_ptr(),
                                      meta.data_ptr() + 8, ws.data_ptr(), ws.numel(),
                                      torch.cuda.current_stream().cuda_stream) == 0
    got = _kernels(run)
    print("decode launches", kind, S, nbytes, s.numel(), got, flush=True)
    assert got == most
    assert out.cpu().numpy().tobytes() == x.tobytes()
    bd = gpulz.BatchDecompressor([s], [nbytes])
    assert _kernels(bd.run) == most + 2
