"""The tuner times a chunk size and window once where the encoder does not use the
waves per chunk, and every number of waves where it does."""
import pytest

from paper_2304_07342_amd import autotune


@pytest.mark.parametrize("S,min_match,chunks,times", [(1, 2, (4096,), 1), (2, 3, (8192,), 1), (1, 1, (4096,), 2),
                                                      (4, 2, (8192,), 1), (4, 2, (12288,), 2), (8, 2, (4096,), 1)])
def test_each_kernel_is_timed_once(monkeypatch, S, min_match, chunks, times):
    calls = []

    def measure(sample, S, C, W, min_match, waves, reps):
        calls.append((C, W, waves))
        return 1.0 + len(calls), 2.0
    monkeypatch.setattr(autotune, "measure", measure)

    class Sample:
        def numel(self):
            return 1000
    got = autotune.tune_width(Sample(), S, min_match, cands=autotune.candidates(S, chunks=chunks, windows=(64, 128)))
    assert len(calls) == 2 * times and len(got["measurements"]) == len(calls)
    assert (got["chunk_symbols"], got["window"]) == (chunks[0], 64)
