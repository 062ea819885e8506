"""Huffman code construction and chunk decoding at the places where joining
many nodes a round and writing 16 bytes a store can go wrong: equal weights at
every symbol count around a lane group, weights that tie with the sums of
lighter ones, a chain of one join a round, lengths that end anywhere in a
store, and an output with room to spare. Streams are byte-identical to the
oracle's (exact, no tolerance)."""
import numpy as np
import pytest

import oracle
from paper_2304_07342_amd import gpulz

pytestmark = pytest.mark.gpu


def _dev(data):
    import torch
    return torch.from_numpy(np.frombuffer(data, np.uint8).copy()).to("cuda")


def _of_weights(w):
    return b"".join(bytes([s]) * int(c) for s, c in enumerate(w))


def _weights():
    rng = np.random.default_rng(77)
    for m in (2, 3, 5, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256):
        yield f"equal_{m}", [3] * m
    yield "ones_and_sums", [1] * 100 + [2] * 60 + [4] * 40 + [8] * 20 + [16] * 10
    yield "small_256", rng.integers(1, 5, 256)
    yield "sparse", rng.integers(0, 3, 256)
    yield "two_scales", np.where(rng.random(256) < 0.5, 1, 700)
    yield "powers", [1 << (k // 16) for k in range(256)]
    yield "doubling", [1] + [1 << k for k in range(14)]
    fib = [1, 1]
    while len(fib) < 20:
        fib.append(fib[-1] + fib[-2])
    yield "chain", fib
    yield "chain_and_ties", fib[:15] + [1] * 120 + [5] * 100


WEIGHTS = list(_weights())


@pytest.mark.parametrize("name,w", WEIGHTS, ids=[n for n, _ in WEIGHTS])
def test_codes_with_ties(name, w):
    data = _of_weights(w)
    print("huff ties", name, len(data), flush=True)
    ref = oracle.huff_compress(data)
    assert gpulz.huff_compress(_dev(data)).cpu().numpy().tobytes() == ref


@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 18, 31, 33, 127, 130, 4096 + 13, 8 * 4096 + 1,
                               9 * 4096 - 1, 3 * 4096 + 128 * 5 + 6])
def test_ends_inside_a_store(n):
    rng = np.random.default_rng(n)
    data = bytes(np.minimum(rng.geometric(0.05, n), 255).astype(np.uint8))
    print("huff ends", n, flush=True)
    back = gpulz.huff_decompress(_dev(oracle.huff_compress(data)))
    assert back.cpu().numpy().tobytes() == data


def test_nothing_written_past_the_end():
    import torch
    rng = np.random.default_rng(5)
    n = 5 * 4096 + 77
    data = bytes(np.minimum(rng.geometric(0.1, n), 255).astype(np.uint8))
    stream = _dev(oracle.huff_compress(data))
    out = torch.full((n + 40 * 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.empty(gpulz.gpulz_huff_decompress_workspace_size(stream.numel()), dtype=torch.uint8,
                     device="cuda")
    meta = torch.zeros(2, dtype=torch.int64, device="cuda")
    print("huff room to spare", flush=True)
    st = gpulz.gpulz_huff_decompress(stream.data_ptr(), stream.numel(), out.data_ptr(), out.numel(),
                                     meta.data_ptr(), meta.data_ptr() + 8, ws.data_ptr(), ws.numel(),
                                     torch.cuda.current_stream().cuda_stream)
    assert st == 0 and meta.tolist() == [n, 0]
    host = out.cpu().numpy()
    assert host[:n].tobytes() == data
    assert (host[n:] == 0xA5).all()


def test_weights_past_32_bits():
    """2 GiB and more: the tree is built on 64-bit weights. Code lengths
    against the reference's, and the chunks read back."""
    import torch
    import huffref
    n = (1 << 31) + 54321
    freq = [0] * 256
    left = n
    for s in range(0, 40, 2):
        freq[s] = left // 3
        left -= freq[s]
    freq[255] = left
    x = torch.empty(n, dtype=torch.uint8, device="cuda")
    at = 0
    for s, c in enumerate(freq):
        x[at:at + c] = s
        at += c
    assert at == n
    print("huff past 32 bits", flush=True)
    stream = gpulz.huff_compress(x)
    packed = stream[64:192].cpu().numpy()
    got = [int(packed[s // 2] >> (4 * (s & 1))) & 15 for s in range(256)]
    assert got == list(huffref.lengths(freq))
    assert torch.equal(gpulz.huff_decompress(stream), x)
