"""gk_verify of pairs that cannot be compared among ones that can: windows past
the reference end and unknown bases at the head of every tile's list (the
longest reads under the largest threshold are computed first), where the
tile's other pairs, and its last, partly filled wave above all, must keep
their distances.  Without accept codes every pair is listed."""
import numpy as np
import pytest

import oracle
from gpu_cases import concat_reads, say
from paper_2103_14978_amd import device, gk
from test_gpu_verify_forms import distances

pytestmark = pytest.mark.gpu


def some_pairs(rng, ref, kinds, m):
    """kinds pairs (read i with window i): reads, offsets, positions, e and the
    expected distances."""
    seqs, pos, e = [], [], []
    for k in range(kinds):
        if k % 16 == 0:                        # longest read, largest threshold, not comparable
            p, s = len(ref) - m // 2, bytearray(ref[-m:].tobytes())
            if k % 32:
                p = int(rng.integers(0, len(ref) - 2 * m))
                s = bytearray(ref[p:p + m].tobytes())
                s[int(rng.integers(0, m))] = ord("N")
            seqs.append(bytes(s))
            e.append(31)
        else:
            n = int(rng.integers(20, m + 1))
            p = int(rng.integers(20, len(ref) - 2 * m))
            s = ref[p + k % 5 - 2:p + k % 5 - 2 + n].copy()
            s[rng.random(n) < 0.06] = ord("G")
            seqs.append(s.tobytes())
            e.append(int(rng.integers(0, 34)))
        pos.append(p)
    reads, off = concat_reads(seqs)
    pos, e = np.array(pos, np.uint32), np.array(e, np.uint8)
    want = np.full(kinds, gk.GK_EST_NONE, np.uint16)
    idx = np.arange(kinds, dtype=np.uint32)
    for t in range(32):
        sel = np.nonzero((e == t) & (idx % 16 != 0))[0]
        want[sel] = oracle.levenshtein_batch(reads, off, ref, idx[sel], pos[sel], t, n_threads=8)
    return reads, off, pos, e, want


# tiles of 256, 512, 1024 and 2048 pairs; furthest-reaching points and bands
@pytest.mark.parametrize("m", [100, 250])
@pytest.mark.parametrize("n", [1000, (1 << 17) + 77, (1 << 19) + 300, (3 << 18) + 1000])
def test_pairs_that_cannot_be_compared(gkctx, n, m):
    rng = np.random.default_rng(n + m)
    ref = rng.choice(np.frombuffer(b"ACGT", np.uint8), 300_000)
    gk.gk_load_reference(gkctx, ref)
    reads, off, pos, e, want = some_pairs(rng, ref, 6000, m)
    dr = device.encode_reads(gkctx, reads, off, max_len=m)
    pick = rng.integers(0, len(pos), n).astype(np.uint32)
    codes = rng.choice(np.array([gk.GK_ACCEPT, gk.GK_REJECT], np.uint8), n, p=[0.7, 0.3])
    for accept in (None, codes):
        say(f"case: verify gate n={n} m={m} codes={accept is not None}")
        got = distances(gkctx, dr, pick, pos[pick], e[pick], accept)
        exp = want[pick]
        if accept is not None:
            exp = np.where(accept == gk.GK_ACCEPT, exp, gk.GK_EST_NONE)
        bad = np.nonzero(got != exp)[0]
        assert len(bad) == 0, (f"{len(bad)} of {n} differ; first {bad[0]}: {got[bad[0]]} for "
                               f"{exp[bad[0]]}")
