"""gk_tune_mixed times its candidates by the calls that gk_filter_mixed would make:
the sampled pairs' results are those of the batch's semantics."""
import json

import pytest

import gen
import oracle
from gpu_cases import assert_same, say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [gk.GK_FLAG_NO_REFINE, gk.GK_FLAG_HAMMING_FASTPATH])
@pytest.mark.parametrize("n", [20_000, 60_000])
def test_tuner_keeps_the_batch_semantics(gkctx, n, flags):
    import torch
    ref = gen.reference(3_000_000, gen.GC_HUMANLIKE, 919)
    gk.gk_load_reference(gkctx, ref)
    ps = gen.pairs(ref, seed=74, n_reads=n // 3, lengths=[100, 150, 300], cand_kind=gen.CAND_GEOM,
                   cand_param=1 / 4, cand_cap=16, true_frac=0.5, edit_kind=gen.EDIT_RATE,
                   edit_param=1.2, e_frac=0.12, band_cands=True)
    assert ps.n_pairs >= n
    want = oracle.filter_batch(ps.reads, ps.read_off, ref, ps.pair_read[:n], ps.cand_pos[:n],
                               ps.e[:n], flags=flags, n_threads=8)
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=300)
    dp = device.upload_pairs(ps.pair_read[:n], ps.cand_pos[:n], ps.e[:n])
    dp.accept.fill_(0xEE)
    dp.est.fill_(0x5A5A)
    say(f"case: tuner flags={flags} n={n}")
    rep = json.loads(gk.gk_tune_mixed(gkctx, device.batch_for(dr, dp, max_read_len=300,
                                                              flags=flags), None))
    torch.cuda.synchronize()
    for opt, val in ((gk.GK_OPT_MIXED_TILE, 4096), (gk.GK_OPT_MIXED_PAIRS_PER_LANE, 1),
                     (gk.GK_OPT_MIXED_SORT_E, 1), (gk.GK_OPT_MIXED_BLOCKS_PER_CU, 0)):
        gk.gk_set_option(gkctx, opt, val)
    assert rep["source"] == "measured"
    a, s = device.results(dp)
    assert_same(a, s, *want, f"tuned flags={flags}")
