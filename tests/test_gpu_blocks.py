"""Reads that just fill, and just overfill, the words that overlap by two bits
in every 64 (62 positions to a block of two words, 30 to a last single word),
at thresholds on both sides of the 30 shifts those words are used for."""
import numpy as np
import pytest

from gpu_cases import assert_same, concat_reads, run_gpu, run_oracle, say
from paper_2103_14978_amd import gk

pytestmark = pytest.mark.gpu


def capacity(words):
    return 32 * words - 2 * ((words - 1) // 2)


@pytest.mark.parametrize("words", [1, 2, 3, 4, 5, 7, 8, 10, 15, 16])
def test_reads_at_a_block_words_end(gkctx, words):
    rng = np.random.default_rng(7100 + words)
    ref = np.full(30_000, ord("A"), np.uint8)
    at = rng.random(30_000) < 1 / 5
    ref[at] = rng.choice(np.frombuffer(b"CGT", np.uint8), int(at.sum()))
    gk.gk_load_reference(gkctx, ref)
    cap = capacity(words)
    lengths = sorted({32 * (words - 1) + 1, cap - 2, cap - 1, cap, min(cap + 1, 32 * words)})
    seqs, pos = [], []
    for i in range(256):
        m, p = lengths[i % len(lengths)], int(rng.integers(40, 29_000))
        s = ref[p + i % 9 - 4:p + i % 9 - 4 + m].copy()
        s[rng.random(m) < 0.06] = ord("G")
        seqs.append(s.tobytes())
        pos.append(p)
    reads, off = concat_reads(seqs)
    pr, pos = np.arange(256, dtype=np.uint32), np.array(pos, np.uint32)
    for e in (0, 1, 2, 5, 29, 30, 31):
        say(f"case: block words={words} e={e}")
        want = run_oracle(ref, reads, off, pr, pos, e)
        a, s, _ = run_gpu(gkctx, ref, reads, off, pr, pos, e, max_read_len=max(lengths),
                          load_ref=False)
        assert_same(a, s, *want, f"block words={words} e={e}")
