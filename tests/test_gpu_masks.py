"""Mask edges: reads and windows made mostly of one base, so that runs of
matches cross the ends of the read, the vacated positions (code 00, the code
of A) and the ends of 32-base words, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_cases import assert_same, concat_reads, run_gpu, run_oracle, say
from paper_2103_14978_amd import gk

pytestmark = pytest.mark.gpu


def runs_of_a(rng, n):
    """n bases, A but for one in six."""
    s = np.full(n, ord("A"), np.uint8)
    at = rng.random(n) < 1 / 6
    s[at] = rng.choice(np.frombuffer(b"CGT", np.uint8), int(at.sum()))
    return s


@pytest.mark.parametrize("m", [1, 2, 3, 31, 32, 33, 34, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160,
                               192, 224, 250, 256, 257, 288, 320, 352, 416, 512])
def test_runs_at_the_edges(gkctx, m):
    rng = np.random.default_rng(900 + m)
    ref = runs_of_a(rng, 40_000)
    gk.gk_load_reference(gkctx, ref)
    seqs, pos = [], []
    for i in range(192):
        p = int(rng.integers(40, 40_000 - m - 40))
        if i % 3 == 0:
            s = runs_of_a(rng, m)
        else:
            s = ref[p + i % 7 - 3:p + i % 7 - 3 + m].copy()
            s[rng.random(m) < 0.05] = ord("C")
        seqs.append(s.tobytes())
        pos.append(p)
    reads, off = concat_reads(seqs)
    pr, pos = np.arange(192, dtype=np.uint32), np.array(pos, np.uint32)
    for e in sorted({0, 1, 2, 3, 15, 30, 31, 32, 33, 64, m - 1, m // 10} & set(range(256))):
        want = run_oracle(ref, reads, off, pr, pos, e)
        for words in {(m + 31) // 32, 16}:      # words just filled, and words left empty
            say(f"case: runs m={m} e={e} words={words}")
            a, s, _ = run_gpu(gkctx, ref, reads, off, pr, pos, e,
                              max_read_len=m if words < 16 else 512, load_ref=False)
            assert_same(a, s, *want, f"runs m={m} e={e} words={words}")
