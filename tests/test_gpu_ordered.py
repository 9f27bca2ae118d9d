"""The plain call with a threshold per pair on batches that need no sort: tiles
whose thresholds and lengths lie in runs are left in order, others are sorted,
at each width of that form's kernels.  Every pair against the plain kernel (one
pair per lane asked for by option) and a sample against the oracle."""
import numpy as np
import pytest

import gen
from gpu_cases import assert_same, run_oracle, say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ref():
    r = gen.reference(3_000_000, gen.GC_HUMANLIKE, 717)
    r[1_000_000:1_002_000] = ord("N")
    return r


def thresholds(kind, n, m):
    i = np.arange(n)
    if kind == "constant":
        return np.full(n, 3, np.uint8)
    if kind == "far":                       # more than 31 shifts, the general path
        return np.full(n, 33, np.uint8)
    if kind == "runs of 64":
        return (i // 64 % 7).astype(np.uint8)
    if kind == "one tile differs":          # the others stay in order
        e = np.full(n, 5, np.uint8)
        e[4096 + 77] = 9
        e[8192:8192 + 64] = 40
        return e
    return (i // 96 % (m // 10)).astype(np.uint8)      # runs across the 64


@pytest.mark.parametrize("kind", ["constant", "far", "runs of 64", "one tile differs",
                                  "runs of 96"])
@pytest.mark.parametrize("lengths", [(150,), (100, 190), (250,), (300,), (330, 370), (500,)],
                         ids=lambda v: "x".join(map(str, v)))
def test_thresholds_in_runs(gkctx, ref, lengths, kind):
    import torch
    gk.gk_load_reference(gkctx, ref)
    layout = gk.GK_READS_INTERLEAVED if kind == "runs of 64" else gk.GK_READS_SPLIT
    n = (1 << 18) + 77 if lengths != (250,) else (1 << 19) + 300
    ps = gen.pairs(ref, seed=65, n_reads=n // 4, lengths=list(lengths), cand_kind=gen.CAND_GEOM,
                   cand_param=1 / 5, cand_cap=16, true_frac=0.5, edit_kind=gen.EDIT_RATE,
                   edit_param=1.2, e_frac=0.05)
    ps.reads[ps.read_off[::97][:-1]] = ord("N")
    assert ps.n_pairs >= n
    e = thresholds(kind, n, max(lengths))
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=max(lengths), layout=layout)
    outs = []
    for ppl in (0, 1):
        dp = device.upload_pairs(ps.pair_read[:n], ps.cand_pos[:n], e, with_bits=True)
        dp.accept_bits.fill_(-1)
        gk.gk_set_option(gkctx, gk.GK_OPT_PAIRS_PER_LANE, ppl)
        say(f"case: thresholds in runs {lengths} {kind} ppl={ppl}")
        gk.gk_filter(gkctx, device.batch_for(dr, dp), None)
        torch.cuda.synchronize()
        outs.append(device.results(dp) + (dp.accept_bits.cpu().numpy(),))
    gk.gk_set_option(gkctx, gk.GK_OPT_PAIRS_PER_LANE, 0)
    assert_same(outs[0][0], outs[0][1], outs[1][0], outs[1][1], kind)
    assert np.array_equal(outs[0][2], outs[1][2])
    some = np.concatenate([np.arange(300), np.arange(4096, 4296), np.arange(8150, 8350),
                           np.arange(n - 200, n)])
    want = run_oracle(ref, ps.reads, ps.read_off, ps.pair_read[some], ps.cand_pos[some], e[some])
    assert_same(outs[0][0][some], outs[0][1][some], *want, f"{kind}, oracle")
