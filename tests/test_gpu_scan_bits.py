"""GPU parity of the policy-1 walk over masks of 32 equal slots (MIN >= 2): runs
of one symbol that pass over the next slot, in stretches of equal slots of every
length and across the masks' edges, windows that are not a multiple of 32, long
runs, the 255 cap, the chunk's start and end. Byte-equal to the oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_compress, gpu_decompress
from paper_2304_07342_amd import gpulz, synth
from test_gpu_bucket import repeats
from test_gpu_wide import planted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 4, 8])
@pytest.mark.parametrize("kind", ["few", "stretches", "runs", "repeats"])
def test_scan_masks(S, kind):
    for C in (33, 400, 1300, 4096):
        m = 2 * C + C // 2
        if kind == "few":
            x = synth.small_alphabet(m, S, C, alphabet=3)
        elif kind == "stretches":  # stretches of 1..70 equal symbols, then one other
            rng = np.random.default_rng(C)
            parts = [np.r_[np.full(int(rng.integers(1, 70)), 7), int(rng.integers(3, 10))] for _ in range(m)]
            x = np.concatenate(parts)[:m].astype({1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}[S]).view(np.uint8)
        elif kind == "runs":
            x = synth.runs(m, S, C)
        else:
            x = repeats(m, S, C, 6) if S <= 2 else planted(m, S, C, 100, 60, C)
        for W, MIN in ((1, 2), (31, 2), (32, 2), (33, 3), (127, 2), (130, 2), (256, 4)):
            print("scan masks", S, kind, C, W, MIN, flush=True)
            st, s, _, canary = gpu_compress(x, S, C, W, MIN, policy=1)
            assert st == gpulz.GPULZ_OK and canary
            assert s == oracle.compress(x, S, C, W, MIN, policy=1)
            st, d, _, canary = gpu_decompress(s, x.size)
            assert st == gpulz.GPULZ_OK and canary and d == x.tobytes()
