"""accept_bits of small batches whose pairs share lanes: the bitmap is a view
inside a larger buffer, and the words around its ceil(n / 64) stay as they
were.  With two lanes per pair a workgroup covers two words of the bitmap, so
an odd number of words ends inside one."""
import numpy as np
import pytest

import gen
from gpu_cases import assert_same, run_oracle, say
from paper_2103_14978_amd import device, gk

pytestmark = pytest.mark.gpu

GUARD = 0x5A5A5A5A5A5A5A5A
CALLS = {"gk_filter": gk.gk_filter, "gk_filter_mixed": gk.gk_filter_mixed,
         "gk_filter_mixed_noalloc": gk.gk_filter_mixed_noalloc}


@pytest.fixture(scope="module")
def ref():
    r = gen.reference(2_000_000, gen.GC_HUMANLIKE, 616)
    r[900_000:901_000] = ord("N")
    return r


# (read length, threshold or one per pair) of two lanes per pair from 24,577
# pairs on, of eight and four below that
@pytest.mark.parametrize("m,e", [(250, 25), (200, None), (128, 31)])
def test_words_around_the_bitmap(gkctx, ref, m, e):
    import torch
    gk.gk_load_reference(gkctx, ref)
    n_max = 49_152
    ps = gen.pairs(ref, seed=64, n_reads=n_max, lengths=[m], true_frac=0.5,
                   edit_kind=gen.EDIT_RATE, edit_param=1.2, e_frac=0.12)
    assert ps.n_pairs == n_max
    ev = ps.e if e is None else np.full(n_max, e, np.uint8)
    want = run_oracle(ref, ps.reads, ps.read_off, ps.pair_read, ps.cand_pos, ev)
    dr = device.encode_reads(gkctx, ps.reads, ps.read_off, max_len=m)
    text = torch.from_numpy(np.concatenate([ps.reads, np.zeros(64, np.uint8)])).cuda()
    off = torch.from_numpy(ps.read_off.view(np.int64)).cuda()
    for n in (1, 64, 12_288, 12_289, 24_576, 24_577, 24_640, 24_641, 40_000, 49_089, 49_152):
        words = (n + 63) // 64
        for name in [*CALLS, "gk_filter_ascii"]:
            say(f"case: bitmap bounds m={m} e={e} n={n} {name}")
            around = torch.full((words + 16,), GUARD, dtype=torch.int64, device="cuda")
            dp = device.upload_pairs(None, ps.cand_pos[:n], ev[:n] if e is None else None)
            dp.accept_bits = around[8:8 + words]
            b = device.batch_for(dr, dp, e_uniform=e or 0)
            if name == "gk_filter_ascii":
                gk.gk_filter_ascii(gkctx, b, text, off, None)
            else:
                CALLS[name](gkctx, b, None)
            torch.cuda.synchronize()
            a, s = device.results(dp)
            assert_same(a, s, want[0][:n], want[1][:n], f"{name} n={n}")
            got = around.cpu().numpy()
            assert (got[:8] == GUARD).all() and (got[8 + words:] == GUARD).all(), f"{name} n={n}"
            bits = np.unpackbits(got[8:8 + words].copy().view(np.uint8), bitorder="little")
            on = (want[0][:n] == gk.GK_ACCEPT) | (want[0][:n] == gk.GK_UNDEFINED)
            assert np.array_equal(bits[:n].astype(bool), on) and not bits[n:].any(), f"{name} n={n}"
