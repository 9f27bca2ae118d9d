"""gk_verify of batches listed as a whole: small thresholds in one list, and a
threshold per pair in order of (words, e) with the reads copied row by row.
The pairs repeat a few thousand whose distances the oracle gives, pairs that
cannot be compared and thresholds above 31 among them."""
import ctypes

import numpy as np
import pytest

import oracle
from gpu_cases import say
from paper_2103_14978_amd import device, gk
from test_gpu_verify_forms import distances
from test_gpu_verify_gate import some_pairs

pytestmark = pytest.mark.gpu

N = (1 << 22) + 4133


@pytest.fixture(scope="module")
def ref():
    return np.random.default_rng(5).choice(np.frombuffer(b"ACGT", np.uint8), 300_000)


def expected(want, pick, accept):
    exp = want[pick]
    return exp if accept is None else np.where(accept == gk.GK_ACCEPT, exp, gk.GK_EST_NONE)


def check(got, exp, label):
    bad = np.nonzero(got != exp)[0]
    assert len(bad) == 0, f"{label}: {len(bad)} differ; first {bad[0]}: {got[bad[0]]} for {exp[bad[0]]}"


@pytest.mark.parametrize("layout", [gk.GK_READS_SPLIT, gk.GK_READS_INTERLEAVED])
@pytest.mark.parametrize("m", [31, 100, 128, 129, 256, 300, 500])
def test_threshold_per_pair(gkctx, ref, m, layout):
    rng = np.random.default_rng(m)
    gk.gk_load_reference(gkctx, ref)
    reads, off, pos, e, want = some_pairs(rng, ref, 4000, m)
    dr = device.encode_reads(gkctx, reads, off, max_len=m, layout=layout)
    pick = rng.integers(0, len(pos), N).astype(np.uint32)
    codes = rng.choice(np.array([0, 1, 2, 3], np.uint8), N, p=[0.6, 0.2, 0.1, 0.1])
    for accept in (codes, None):
        say(f"case: verify listed m={m} layout={layout} codes={accept is not None}")
        got = distances(gkctx, dr, pick, pos[pick], e[pick], accept)
        check(got, expected(want, pick, accept), f"m={m}")


def small_thresholds(rng, ref, m, e):
    reads, off, pos, _, _ = some_pairs(rng, ref, 3000, m)
    idx = np.arange(len(pos), dtype=np.uint32)
    want = oracle.levenshtein_batch(reads, off, ref, idx, pos, e, n_threads=8)
    want[idx % 16 == 0] = gk.GK_EST_NONE
    return reads, off, pos, want


@pytest.mark.parametrize("m,e", [(64, 0), (100, 5), (250, 7), (300, 3), (512, 7)])
def test_one_small_threshold(gkctx, ref, m, e):
    """Also with buffers that are not 16-byte aligned, and reads of length 0
    and above max_read_len."""
    import torch
    rng = np.random.default_rng(m + e)
    gk.gk_load_reference(gkctx, ref)
    reads, off, pos, want = small_thresholds(rng, ref, m, e)
    dr = device.encode_reads(gkctx, reads, off, max_len=m)
    dr.read_len[5], dr.read_len[6] = 0, m + 1
    want[5] = want[6] = gk.GK_EST_NONE
    pick = rng.integers(0, len(pos), N).astype(np.uint32)
    codes = rng.choice(np.array([0, 1], np.uint8), N, p=[0.9, 0.1])
    for accept in (codes, None):
        for shift in (0, 1):
            say(f"case: verify listed m={m} e={e} codes={accept is not None} shift={shift}")
            dp = device.upload_pairs(pick, pos[pick])
            acc = None
            if accept is not None:
                acc = torch.from_numpy(np.concatenate([np.zeros(shift, np.uint8), accept])).cuda()[shift:]
            dist = torch.full((N + 8,), 0x5A5A, dtype=torch.int16, device="cuda")[shift:shift + N]
            gk.gk_verify(gkctx, device.batch_for(dr, dp, e_uniform=e), acc, dist)
            torch.cuda.synchronize()
            check(dist.cpu().numpy().view(np.uint16), expected(want, pick, accept), f"m={m} e={e}")


@pytest.mark.parametrize("n", [65_536, 65_537])
def test_one_large_threshold(gkctx, ref, n):
    rng = np.random.default_rng(n)
    gk.gk_load_reference(gkctx, ref)
    reads, off, pos, want = small_thresholds(rng, ref, 130, 20)
    dr = device.encode_reads(gkctx, reads, off, max_len=130)
    pick = rng.integers(0, len(pos), n).astype(np.uint32)
    codes = rng.choice(np.array([0, 1], np.uint8), n, p=[0.3, 0.7])
    for accept in (codes, None):
        say(f"case: verify listed e=20 n={n} codes={accept is not None}")
        check(distances(gkctx, dr, pick, pos[pick], 20, accept), expected(want, pick, accept),
              f"e=20 n={n}")


@pytest.mark.parametrize("n,kinds", [((3 << 19) - 1, 3000), (3 << 19, 3000), (3 << 19, 131_072),
                                     (3 << 19, 131_073), (1 << 24, 2_396_745),
                                     (1 << 24, 2_396_746)])
def test_rule_of_candidates_per_read(gkctx, ref, n, kinds):
    """Both sides of the rule's limits: pairs of the batch, pairs per read."""
    rng = np.random.default_rng(n + kinds)
    gk.gk_load_reference(gkctx, ref)
    reads, off, pos, e, want = some_pairs(rng, ref, 3000, 150)
    dr = device.encode_reads(gkctx, np.tile(reads, -(-kinds // 3000)), np.concatenate(
        [off[:-1] + off[-1] * np.uint64(k) for k in range(-(-kinds // 3000))])[:kinds + 1]
        if kinds > 3000 else off, max_len=150)
    pick = rng.integers(0, min(kinds, dr.n_reads), n).astype(np.uint32)
    say(f"case: verify rule n={n} reads={dr.n_reads}")
    got = distances(gkctx, dr, pick, pos[pick % 3000], e[pick % 3000])
    check(got, want[pick % 3000], f"n={n} reads={dr.n_reads}")


@pytest.mark.parametrize("per_pair", [False, True])
def test_without_scratch(ref, per_pair):
    """Where the list cannot be allocated, and under stream capture, the same
    batch takes the tile form."""
    import torch
    rng = np.random.default_rng(9)
    fail_at = gk.lib().gk_detail_fail_alloc
    fail_at.argtypes, fail_at.restype = [ctypes.c_uint64], ctypes.c_int
    ctx = gk.gk_create(0)
    try:
        gk.gk_load_reference(ctx, ref)
        reads, off, pos, e, want = some_pairs(rng, ref, 3000, 100)
        if not per_pair:
            reads, off, pos, want = small_thresholds(rng, ref, 100, 5)
        dr = device.encode_reads(ctx, reads, off, max_len=100)
        pick = rng.integers(0, len(pos), N).astype(np.uint32)
        dp = device.upload_pairs(pick, pos[pick], e[pick] if per_pair else None)
        batch = device.batch_for(dr, dp, e_uniform=5)
        dist = torch.full((N,), 0x5A5A, dtype=torch.int16, device="cuda")

        def result():
            torch.cuda.synchronize()
            got = dist.cpu().numpy().view(np.uint16).copy()
            dist.fill_(0x5A5A)
            return got
        say(f"case: verify without scratch per_pair={per_pair}")
        fail_at(2)                              # the count word, then the list
        gk.gk_verify(ctx, batch, None, dist)
        fail_at(0)
        check(result(), want[pick], "list not allocated")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            gk.gk_verify(ctx, batch, None, dist, torch.cuda.current_stream())
        gk.gk_verify(ctx, batch, None, dist)    # allocates the list
        check(result(), want[pick], "listed")
        for k in range(3):
            graph.replay()
            check(result(), want[pick], f"replay {k}")
            gk.gk_verify(ctx, batch, None, dist)
            check(result(), want[pick], f"listed after replay {k}")
    finally:
        fail_at(0)
        gk.gk_destroy(ctx)
