"""gk_verify's two forms (pairs listed by tile, and one list of the batch for
large batches under one threshold) on the same pairs, and both algorithms of
the tile form, against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from gpu_cases import say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu


def distances(ctx, dr, pr, pos, e, accept=None):
    import torch
    dp = device.upload_pairs(pr, pos, None if np.isscalar(e) else e)
    acc = None if accept is None else torch.from_numpy(accept).cuda()
    dist = torch.full((len(pos),), 0x5A5A, dtype=torch.int16, device="cuda")
    gk.gk_verify(ctx, device.batch_for(dr, dp, e_uniform=e if np.isscalar(e) else 0), acc, dist)
    torch.cuda.synchronize()
    return dist.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("e,n", [(7, 2049), (8, (1 << 19) + 3), (12, (1 << 18) + 1),
                                 (17, (1 << 17) + 70), (31, 1 << 17)])
def test_list_and_tile_forms_agree(gkctx, e, n):
    """The threshold as an array takes the tile form, as one number the list."""
    ref = gen.c1_reference(4_000_000)
    gk.gk_load_reference(gkctx, ref)
    ps = gen.c2_pairs(ref, 130, e, n_pairs=n)
    n = ps.n_pairs
    rng = np.random.default_rng(e)
    accept = rng.integers(0, 4, n).astype(np.uint8)
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=130)
    say(f"case: verify forms e={e} n={n}")
    a = distances(gkctx, dr, ps.pair_read, ps.cand_pos, e, accept)
    b = distances(gkctx, dr, ps.pair_read, ps.cand_pos, np.full(n, e, np.uint8), accept)
    assert np.array_equal(a, b)
    some = rng.choice(n, min(n, 3000), replace=False)
    want = oracle.levenshtein_batch(ps.reads, ps.read_off, ref, ps.pair_read[some],
                                    ps.cand_pos[some], e, n_threads=8)
    want[accept[some] != gk.GK_ACCEPT] = gk.GK_EST_NONE
    assert np.array_equal(a[some], want)


@pytest.mark.parametrize("m", [1, 2, 31, 32, 33, 64, 100, 127, 128, 129, 320, 512])
def test_small_thresholds_at_word_edges(gkctx, m):
    """Furthest-reaching points with runs over many words and reads no longer
    than the threshold, next to the banded form in one batch."""
    rng = np.random.default_rng(m)
    ref = np.full(20_000, ord("A"), np.uint8)
    at = rng.random(20_000) < 0.02
    ref[at] = rng.choice(np.frombuffer(b"CGT", np.uint8), int(at.sum()))
    gk.gk_load_reference(gkctx, ref)
    pos = rng.integers(40, 20_000 - m - 40, 700).astype(np.uint32)
    reads = np.stack([ref[p + k % 11 - 5:p + k % 11 - 5 + m] for k, p in enumerate(pos)]).copy()
    swap = rng.random(reads.shape) < 0.02
    reads[swap] = ord("G")
    off = np.arange(len(pos) + 1, dtype=np.uint64) * np.uint64(m)
    dr = device.encode_reads(gkctx, reads.reshape(-1), off, max_len=m)
    pr = np.arange(len(pos), dtype=np.uint32)
    e = (np.arange(len(pos)) % 13).astype(np.uint8)
    say(f"case: verify small thresholds m={m}")
    got = distances(gkctx, dr, pr, pos, e)
    for k in range(13):
        sel = np.nonzero(e == k)[0]
        want = oracle.levenshtein_batch(reads.reshape(-1), off, ref, pr[sel], pos[sel], k,
                                        n_threads=8)
        assert np.array_equal(got[sel], want), f"m={m} e={k}"
