"""GPU parity of 1- and 2-byte symbols with MIN >= 3 on match-dense input. The
general encoder once gave up the hit bitmap after a dense first block without
taking the streaming parse in its place, so that every later match was lost:
in launches of more than 1024 chunks, in chunks of more than 4096 symbols and in
batches, with one wave per chunk. Streams must equal the oracle's byte for
byte in every launch form, whatever the waves per chunk."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, to_device
from paper_2304_07342_amd import gpulz
from test_gpu_dense import dense_mix

pytestmark = pytest.mark.gpu


def dense(m: int, S: int, seed: int) -> np.ndarray:
    """m symbols that are match-dense throughout."""
    return np.tile(dense_mix(1 << 14, S, seed), -(-m >> 14))[: m * S]


@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("C,N", [(1300, 1100), (2048, 1025), (4097, 3), (8192, 40), (9000, 3)])
def test_single(S, C, N):
    x = dense((N - 1) * C + C // 3, S, C)
    for W, MIN in ((256, 3), (100, 6)):
        want = oracle.compress(x, S, C, W, MIN, threads=16)
        for waves in (1, 4) if C > 8192 else (1,):
            saved = gpulz.gpulz_default_params(S)
            gpulz.gpulz_set_default_params(S, saved[0], saved[1], saved[2], waves)
            try:
                print("min3", S, C, N, W, MIN, waves, flush=True)
                st, s, _, canary = gpu_compress(x, S, C, W, MIN)
            finally:
                gpulz.gpulz_set_default_params(S, *saved)
            assert st == gpulz.GPULZ_OK and canary and s == want


def test_batch():
    import torch
    params = {1: (4096, 256, 3, 1), 2: (9000, 128, 4, 1)}
    xs = [dense(n, S, 9 + n) for n, S in ((20000, 1), (30001, 2), (4096, 1), (9001, 2))]
    widths = [1, 2, 1, 2]
    bc = gpulz.BatchCompressor([to_device(x)[: x.size] for x in xs], widths, params)
    print("min3 batch", flush=True)
    bc.run()
    torch.cuda.synchronize()
    for (st, s), x, S in zip(bc.results(), xs, widths):
        assert st == gpulz.GPULZ_OK
        assert s.cpu().numpy().tobytes() == oracle.compress(x, S, *params[S][:3])
