"""The direct form of the mixed launch at the edges of its tiles, and the
plain call's sorted route, against the oracle and against the plain kernel."""
import numpy as np
import pytest

import gen
from gpu_cases import assert_same, run_gpu_mixed, run_oracle, say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ref():
    r = gen.reference(3_000_000, gen.GC_HUMANLIKE, 515)
    r[1_000_000:1_002_000] = ord("N")
    return r


def pairs_of(ref, lengths, n_reads, seed, e_frac=0.12):
    ps = gen.pairs(ref, seed=seed, n_reads=n_reads, lengths=lengths, cand_kind=gen.CAND_GEOM,
                   cand_param=1 / 4, cand_cap=16, true_frac=0.5, edit_kind=gen.EDIT_RATE,
                   edit_param=1.2, e_frac=e_frac, band_cands=True)
    ps.reads[ps.read_off[::97][:-1]] = ord("N")
    return ps


@pytest.mark.parametrize("lengths", [(64, 100, 128), (64, 100, 150, 200, 250, 300), (33, 400, 512)],
                         ids=lambda v: f"max{max(v)}")
def test_direct_tile_edges(gkctx, ref, lengths):
    gk.gk_load_reference(gkctx, ref)
    ps = pairs_of(ref, list(lengths), 12_000, 61)
    want = run_oracle(ref, ps.reads, ps.read_off, ps.pair_read, ps.cand_pos, ps.e)
    for n in (1, 65, 5000, 24576, 24577, 24833, 25000):
        say(f"case: direct mixed {max(lengths)} n={n}")
        a, s, bits = run_gpu_mixed(gkctx, ps.reads, ps.read_off, ps.pair_read[:n], ps.cand_pos[:n],
                                   ps.e[:n], max_read_len=max(lengths), with_bits=True)
        assert_same(a, s, want[0][:n], want[1][:n], f"direct n={n}")
        got = np.unpackbits(bits.view(np.uint8), bitorder="little")
        on = (want[0][:n] == 1) | (want[0][:n] == 2)
        assert np.array_equal(got[:n].astype(bool), on) and not got[n:].any()


@pytest.mark.parametrize("layout", [gk.GK_READS_SPLIT, gk.GK_READS_INTERLEAVED])
@pytest.mark.parametrize("identity", [False, True])
@pytest.mark.parametrize("flags_known", [False, True])
def test_plain_call_sorted_route(gkctx, ref, layout, identity, flags_known):
    """2^18 pairs and up with a threshold per pair are sorted; one pair per
    lane asked for by option takes the plain kernel on the same batch."""
    import torch
    gk.gk_load_reference(gkctx, ref)
    n = (1 << 18) + 77
    ps = pairs_of(ref, [90, 150, 300], n + 500 if identity else n // 3, 62)
    assert ps.n_pairs >= n
    pr = None if identity else ps.pair_read[:n]
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=300, layout=layout)
    if not flags_known:
        dr.has_n = None
    outs = []
    for ppl in (0, 1):
        dp = device.upload_pairs(pr, ps.cand_pos[:n], ps.e[:n], with_bits=True)
        dp.accept_bits.fill_(-1)
        gk.gk_set_option(gkctx, gk.GK_OPT_PAIRS_PER_LANE, ppl)
        say(f"case: plain call layout={layout} identity={identity} ppl={ppl}")
        gk.gk_filter(gkctx, device.batch_for(dr, dp), None)
        torch.cuda.synchronize()
        outs.append(device.results(dp) + (dp.accept_bits.cpu().numpy(),))
    gk.gk_set_option(gkctx, gk.GK_OPT_PAIRS_PER_LANE, 0)
    assert_same(outs[0][0], outs[0][1], outs[1][0], outs[1][1], "sorted vs plain")
    assert np.array_equal(outs[0][2], outs[1][2])


@pytest.mark.parametrize("lengths,e", [((100,), None), ((150,), 7), ((250,), 25), ((33, 200, 320), None),
                                       ((64, 500, 512), None)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"e{v}")
def test_lanes_per_pair(gkctx, ref, lengths, e):
    """Small batches share a pair's masks among 8, 4 or 2 lanes: batch sizes at
    and around the rule's limits, and accept bits of partly filled words."""
    import torch
    gk.gk_load_reference(gkctx, ref)
    ps = pairs_of(ref, list(lengths), 25_000, 63, e_frac=0.12)
    ev = ps.e if e is None else np.full(ps.n_pairs, e, np.uint8)
    want = run_oracle(ref, ps.reads, ps.read_off, ps.pair_read, ps.cand_pos, ev)
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=max(lengths))
    text = torch.from_numpy(np.concatenate([ps.reads, np.zeros(64, np.uint8)])).cuda()
    off = torch.from_numpy(ps.read_off.view(np.int64)).cuda()
    first = np.unique(ps.pair_read, return_index=True)[1]     # one candidate per read
    for n in (1, 7, 63, 65, 12288, 12289, 24576, 24577, 49152, 49153):
        if n <= ps.n_pairs:
            say(f"case: lanes {lengths} e={e} n={n}")
            dp = device.upload_pairs(ps.pair_read[:n], ps.cand_pos[:n],
                                     ev[:n] if e is None else None, with_bits=True)
            dp.accept_bits.fill_(-1)
            gk.gk_filter(gkctx, device.batch_for(dr, dp, e_uniform=e or 0), None)
            torch.cuda.synchronize()
            check(dp, want[0][:n], want[1][:n], f"plain n={n}")
        if n <= len(first):
            sel = first[:n]
            dp = device.upload_pairs(None, ps.cand_pos[sel], ev[sel] if e is None else None,
                                     with_bits=True)
            dp.accept_bits.fill_(-1)
            gk.gk_filter_ascii(gkctx, device.batch_for(dr, dp, e_uniform=e or 0), text, off, None)
            torch.cuda.synchronize()
            check(dp, want[0][sel], want[1][sel], f"ascii n={n}")


def check(dp, accept, est, label):
    a, s = device.results(dp)
    assert_same(a, s, accept, est, label)
    got = np.unpackbits(dp.accept_bits.cpu().numpy().view(np.uint8), bitorder="little")
    n = len(accept)
    assert np.array_equal(got[:n].astype(bool), (accept == 1) | (accept == 2)), label
    assert not got[n:].any(), label
