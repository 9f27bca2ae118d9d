"""gk_verify of a large batch, whose tiles grow to 4096 or 8192 pairs by the
words of the longest read, against the same pairs in batches of small tiles and
a sample of them against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from gpu_cases import say
from paper_2103_14978_amd import device, gk
from test_gpu_verify_forms import distances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [200, 300])       # 7 words: 4096 pairs, 10 words: 8192
def test_large_batches_agree_with_small(gkctx, m):
    ref = gen.c1_reference(2_000_000)
    gk.gk_load_reference(gkctx, ref)
    rng = np.random.default_rng(m)
    reads_n, n = 3000, (1 << 22) + 8191
    lens = rng.integers(m // 2, m + 1, reads_n)
    lens[0] = m
    start = rng.integers(10, len(ref) - 400, reads_n)
    seqs = [ref[p:p + k].copy() for p, k in zip(start, lens)]
    for s in seqs:
        s[rng.random(len(s)) < 0.03] = ord("G")
    reads = np.concatenate(seqs)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    pr = rng.integers(0, reads_n, n).astype(np.uint32)
    pos = (start[pr] + rng.integers(-3, 4, n)).astype(np.uint32)
    e = rng.integers(0, 33, n).astype(np.uint8)
    accept = rng.integers(0, 4, n).astype(np.uint8)
    dr = device.encode_reads(gkctx, reads, off, max_len=m)
    say(f"case: verify large tiles m={m}")
    got = distances(gkctx, dr, pr, pos, e, accept)
    for a, b in ((0, 100_000), (2_000_000, 2_100_000), (n - 100_000, n)):
        part = distances(gkctx, dr, pr[a:b], pos[a:b], e[a:b], accept[a:b])
        assert np.array_equal(got[a:b], part), f"pairs {a} to {b}"
    some = rng.choice(np.nonzero((accept == gk.GK_ACCEPT) & (e == 20))[0], 1000, replace=False)
    want = oracle.levenshtein_batch(reads, off, ref, pr[some], pos[some], 20, n_threads=8)
    assert np.array_equal(got[some], want)
    assert (got[accept != gk.GK_ACCEPT] == gk.GK_EST_NONE).all()
    assert (got[e > 31] == gk.GK_EST_NONE).all()
