"""The forms of the mixed launch that only some batches reach: the captured one
(a tuning set, fewer tiles than compute units) with its ring of pinned argument
tables, the direct one at up to 4 words per mask, and the sort on batches that
the default tuning would leave unsorted.  Every pair against the oracle."""
import numpy as np
import pytest

import gen
from gpu_cases import assert_same, run_gpu_mixed, run_oracle, say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu

TUNED = {gk.GK_OPT_MIXED_TILE: 8192}          # 2048 pairs per tile


@pytest.fixture(scope="module")
def ref():
    r = gen.reference(3_000_000, gen.GC_HUMANLIKE, 818)
    r[1_000_000:1_002_000] = ord("N")
    return r


def make_pairs(ref, lengths, n, seed, e_frac=0.12):
    ps = gen.pairs(ref, seed=seed, n_reads=n // 3, lengths=lengths, cand_kind=gen.CAND_GEOM,
                   cand_param=1 / 4, cand_cap=16, true_frac=0.5, edit_kind=gen.EDIT_RATE,
                   edit_param=1.2, e_frac=e_frac, band_cands=True)
    ps.reads[ps.read_off[::97][:-1]] = ord("N")
    assert ps.n_pairs >= n
    return ps, run_oracle(ref, ps.reads, ps.read_off, ps.pair_read, ps.cand_pos, ps.e)


def check_bits(bits, accept, label):
    got = np.unpackbits(bits.view(np.uint8), bitorder="little")
    n = len(accept)
    assert np.array_equal(got[:n].astype(bool), (accept == 1) | (accept == 2)), label
    assert not got[n:].any(), label


@pytest.mark.parametrize("lengths", [(64, 128), (64, 150, 300), (33, 400, 512)],
                         ids=lambda v: f"max{max(v)}")
def test_captured_form(gkctx, ref, lengths):
    """Batches of other sizes and buffers replay one graph, eight calls queued
    without a wait between them (the ring holds four argument tables), twice."""
    import torch
    gk.gk_load_reference(gkctx, ref)
    ps, want = make_pairs(ref, list(lengths), 60_000, 71)
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=max(lengths))
    jobs = []
    for k, n in enumerate((60_000, 1, 4097, 24_576, 50_001, 2048, 63, 33_333)):
        sl = slice(k * 1013 % (ps.n_pairs - n + 1), k * 1013 % (ps.n_pairs - n + 1) + n)
        dp = device.upload_pairs(ps.pair_read[sl], ps.cand_pos[sl], ps.e[sl], with_bits=True)
        jobs.append((sl, dp, device.batch_for(dr, dp, max_read_len=max(lengths))))
    for k, v in TUNED.items():
        gk.gk_set_option(gkctx, k, v)
    try:
        for turn in range(2):
            say(f"case: captured form max={max(lengths)} turn={turn}")
            for _, dp, _ in jobs:
                dp.accept.fill_(0xEE)
                dp.est.fill_(0x5A5A)
                dp.accept_bits.fill_(-1)
            torch.cuda.synchronize()
            for _, _, b in jobs:
                gk.gk_filter_mixed(gkctx, b, None)
            torch.cuda.synchronize()
            for sl, dp, _ in jobs:
                a, s = device.results(dp)
                assert_same(a, s, want[0][sl], want[1][sl], f"{sl} turn {turn}")
                check_bits(dp.accept_bits.cpu().numpy(), want[0][sl], f"{sl} turn {turn}")
    finally:
        gk.gk_set_option(gkctx, gk.GK_OPT_MIXED_TILE, 4096)


@pytest.mark.parametrize("options", [{}, {gk.GK_OPT_MIXED_PAIRS_PER_LANE: 2},
                                     {gk.GK_OPT_MIXED_SORT_E: 0}],
                         ids=["default", "two-pairs", "by-words"])
@pytest.mark.parametrize("layout", [gk.GK_READS_SPLIT, gk.GK_READS_INTERLEAVED])
def test_direct_form_of_short_reads(gkctx, ref, layout, options):
    gk.gk_load_reference(gkctx, ref)
    n = (1 << 18) + 333
    ps, want = make_pairs(ref, [33, 64, 100, 128], n, 72, e_frac=0.3)
    say(f"case: direct short reads layout={layout} {options}")
    a, s, bits = run_gpu_mixed(gkctx, ps.reads, ps.read_off, ps.pair_read[:n], ps.cand_pos[:n],
                               ps.e[:n], max_read_len=128, layout=layout,
                               options={**options, gk.GK_OPT_MIXED_GRAPH: 0}, with_bits=True)
    assert_same(a, s, want[0][:n], want[1][:n], "direct short reads")
    check_bits(bits, want[0][:n], "direct short reads")


@pytest.mark.parametrize("lengths", [(64, 128), (64, 150, 300), (33, 400, 512)],
                         ids=lambda v: f"max{max(v)}")
def test_small_batches_sorted(gkctx, ref, lengths):
    gk.gk_load_reference(gkctx, ref)
    ps, want = make_pairs(ref, list(lengths), 5000, 73, e_frac=0.15)
    for n in (1, 63, 257, 512, 513, 5000):
        say(f"case: small sorted max={max(lengths)} n={n}")
        a, s, bits = run_gpu_mixed(gkctx, ps.reads, ps.read_off, ps.pair_read[:n],
                                   ps.cand_pos[:n], ps.e[:n], max_read_len=max(lengths),
                                   options={gk.GK_OPT_MIXED_TILE: 2048, gk.GK_OPT_MIXED_GRAPH: 0},
                                   with_bits=True)
        assert_same(a, s, want[0][:n], want[1][:n], f"small n={n}")
        check_bits(bits, want[0][:n], f"small n={n}")


@pytest.mark.parametrize("m", [100, 250, 500])
def test_one_large_threshold(gkctx, ref, m):
    """Up to 3 * 2^16 pairs under one threshold above 31 go as they come."""
    gk.gk_load_reference(gkctx, ref)
    n_max = (3 << 16) + 1
    ps = gen.pairs(ref, seed=75, n_reads=n_max // 3, lengths=[m // 2, m], cand_kind=gen.CAND_GEOM,
                   cand_param=1 / 4, cand_cap=16, true_frac=0.5, edit_kind=gen.EDIT_RATE,
                   edit_param=1.2, e_frac=0.12)
    assert ps.n_pairs >= n_max
    e = 33
    want = run_oracle(ref, ps.reads, ps.read_off, ps.pair_read, ps.cand_pos, e)
    for n in (1000, 24_577, 131_073, 3 << 16, n_max):
        say(f"case: one large threshold m={m} n={n}")
        a, s, bits = run_gpu_mixed(gkctx, ps.reads, ps.read_off, ps.pair_read[:n],
                                   ps.cand_pos[:n], e, max_read_len=m, with_bits=True)
        assert_same(a, s, want[0][:n], want[1][:n], f"large threshold n={n}")
        check_bits(bits, want[0][:n], f"large threshold n={n}")
