"""Timed cases of the GateKeeper filter, through the public entry points of
paper_2103_14978_amd.gk.

The inputs stand in for a read mapper's: reads drawn from a genome with
substitutions, insertions and deletions, paired with their origin, with
shifts of it (a seed hit off by an indel), or with unrelated positions that
share an exact 12-mer (a seed's false hit).  The genomes are fixed, as a
mapper loads one and keeps it; reads, positions and thresholds come from the
seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2103_14978_amd import gk

DEV = "cuda:0"
GENOMES = {"chromosome": 100_000_000, "human": 3_100_000_000}
# Read lengths of a batch that mixes several sequencing runs, per-pair
# thresholds 0 .. a tenth of the length.
MIX = (64, 100, 150, 200, 250, 300)


def listed():
    return [
        # The smallest request of a served mapper: launch and call overhead.
        dict(name="filter_100bp_1k", op="filter", genome="chromosome", n=1000, m=100, e=5,
             cands=1, bits=False),
        # One sequencing batch of short reads, one candidate per read.
        dict(name="filter_100bp_16m", op="filter", genome="chromosome", n=1 << 24, m=100, e=5,
             cands=1, bits=False),
        # A whole human genome with its runs of unknown bases, several
        # candidates per read, the accept bitmap a mapper compacts by.
        dict(name="filter_150bp_human", op="filter", genome="human", n=3_000_017, m=150, e=7,
             cands=8, bits=True),
        # Long reads at the largest threshold in use (a tenth of the length).
        dict(name="filter_250bp_e25", op="filter", genome="chromosome", n=1 << 23, m=250, e=25,
             cands=8, bits=False),
        # Reads straight from a FASTQ parser: encoded and filtered in one call.
        dict(name="ascii_100bp_4m", op="ascii", genome="chromosome", n=4_194_301, m=100, e=5,
             cands=1, bits=False),
        # Encoding of reads of several lengths, used for many batches later.
        dict(name="encode_mix_2m", op="encode", genome="chromosome", n=2_000_003, m=0, e=0,
             cands=1, bits=False),
        # Mixed lengths and thresholds in one batch: a large batch ...
        dict(name="mixed_16m", op="mixed", genome="chromosome", n=1 << 24, m=0, e=-1,
             cands=3, bits=False),
        # ... and an ordinary request.
        dict(name="mixed_60k", op="mixed", genome="human", n=60_001, m=0, e=-1, cands=8,
             bits=True),
        # Exact distances of the pairs the filter passed, one length and e.
        dict(name="verify_100bp_4m", op="verify", genome="chromosome", n=1 << 22, m=100, e=5,
             cands=1, bits=False),
        # The same for a mixed batch.
        dict(name="verify_mix_1m", op="verify", genome="chromosome", n=1_048_573, m=0, e=-1,
             cands=3, bits=False),
        # Reads and results in host memory, the whole call.
        dict(name="host_100bp_2m", op="host", genome="chromosome", n=2_097_143, m=100, e=5,
             cands=1, bits=False),
        # A burst of requests of mixed sizes to the batched server.
        dict(name="served_burst", op="served", genome="human", n=1_200_000, m=0, e=-1, cands=8,
             bits=False),
    ]


def _cost(case):
    w = work(case)
    return w["bytes"] / 8e12 + w["flops"] / 39e12


def draw(rng):
    """A case over the same ranges: 1,000 to 2^24 pairs (a tenth of that where
    the data is the host's), reads of 40 to 512 bases or the mix, thresholds
    up to a tenth of the length or per pair."""
    op = rng.choice(["filter"] * 4 + ["ascii"] * 2 + ["encode"] + ["mixed"] * 2 + ["verify"] * 2 +
                    ["host"])
    top = 1 << 21 if op == "host" else 1 << 24
    n = int(math.exp(rng.uniform(math.log(1000), math.log(top))))
    m = 0 if op == "mixed" or rng.random() < 0.2 else int(
        math.exp(rng.uniform(math.log(40), math.log(512))))
    e = 0 if op == "encode" else -1 if m == 0 or rng.random() < 0.15 else rng.randint(0, m // 10)
    e = min(e, gk.GK_VERIFY_MAX_E) if op == "verify" else e
    cands = 1 if op in ("ascii", "encode", "host") else rng.choice([1, 3, 8])
    case = dict(op=op, genome=rng.choice(["chromosome", "human"]), n=n, m=m, e=e, cands=cands,
                bits=op in ("filter", "mixed") and rng.random() < 0.4)
    most = max(_cost(c) for c in listed())
    if _cost(case) > most:
        case["n"] = max(1000, int(n * most / _cost(case)))
    return case


# ----------------------------------------------------------------- genomes ---

_genomes = {}


def _words(n, g):
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device=DEV, dtype=torch.int64).to(
        torch.int32)


def _genome(name):
    """(context, length, packed words, unknown runs) of a genome with 41% GC,
    loaded once; base i is in word i // 16, low code bit at bit i % 16, high
    one at 16 + i % 16 (A C G T = 0 1 2 3, so GC is low != high)."""
    if name not in _genomes:
        length = GENOMES[name]
        g = torch.Generator(device=DEV).manual_seed(1001)
        n = (length + 15) // 16
        hi = _words(n, g) & 0xFFFF
        gc = _words(n, g)                       # P(bit) = 0.40625 = 0.01101b
        for bit in (0, 1, 1, 0):
            x = _words(n, g)
            gc = (gc | x) if bit else (gc & x)
        words = (hi << 16) | ((hi ^ gc) & 0xFFFF)
        runs = None
        if name == "human":
            # 3% of the bases unknown, in runs of 10 kbp to 20 Mbp
            r = np.random.default_rng(1002)
            size = np.exp(r.uniform(np.log(1e4), np.log(2e7), 36)).astype(np.uint64)
            at = r.integers(0, length - 20_000_000, 36).astype(np.uint64)
            runs = np.stack([at, size], 1)
        ctx = gk.gk_create(0)
        gk.gk_load_reference_2bit(ctx, words.cpu().numpy().view(np.uint32), length,
                                  gk.GK_READS_SPLIT, runs)
        _genomes[name] = (ctx, length, words, runs)
    return _genomes[name]


def _bases(words, idx):
    w = words[idx >> 4].to(torch.int32)
    j = (idx & 15).to(torch.int32)
    return ((w >> j) & 1) | (((w >> (16 + j)) & 1) << 1)


# ------------------------------------------------------------------ inputs ---

_LETTERS = (65, 67, 71, 84)          # A C G T


def _batch(case, seed):
    """Reads and pairs of a case on the GPU, as a dict of tensors."""
    _, length, words, _ = _genome(case["genome"])
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)
    n, m, e, cands = case["n"], case["m"], case["e"], case["cands"]

    def rand(*shape):
        return torch.rand(shape, generator=g, device=DEV)

    def below(high, *shape):
        return torch.randint(0, high, shape, generator=g, device=DEV)

    if cands == 1:
        n_reads = n
        pair_read = torch.arange(n, device=DEV)
        rank = None
    else:
        # geometric number of candidates per read, at most 64
        n_reads = max(1, int(n / cands * 1.1) + 64)
        cnt = torch.ceil(torch.log(1 - rand(n_reads)) / math.log(1 - 1 / cands)).clamp(1, 64).long()
        first = torch.cumsum(cnt, 0) - cnt
        pair_read = torch.repeat_interleave(torch.arange(n_reads, device=DEV), cnt)[:n]
        n = pair_read.numel()
        rank = torch.arange(n, device=DEV) - first[pair_read]
    mix = torch.tensor(MIX, device=DEV)
    lens = mix[below(len(MIX), n_reads)] if m == 0 else torch.full((n_reads,), m, device=DEV)
    top = max(MIX) if m == 0 else m
    pair_e = (rand(n) * (lens[pair_read] // 10 + 1)).to(torch.uint8) if e < 0 else None

    span = length - 2 * top - 64
    origin = 32 + (rand(n_reads).double() * span).long()
    true = rand(n_reads) < (0.3 if cands == 1 else 0.45)
    if cands == 1:
        other = 32 + (rand(n_reads).double() * span).long()
        pos = torch.where(true, origin, other)
        shared = other                   # a decoy shares a 12-mer with its window
    else:
        near = (lens // 10)[pair_read] if e < 0 else torch.full_like(pair_read, max(e, 0))
        shift = ((rand(n) * (2 * near + 1)).long() - near)
        away = 32 + (rand(n).double() * span).long()
        pos = origin[pair_read] + torch.where(rank == 0, 0, shift)
        pos = torch.where(true[pair_read] & (rank <= 2 * near), pos, away)
        shared = torch.zeros(n_reads, dtype=torch.int64, device=DEV)
        shared[pair_read[rank == 0]] = pos[rank == 0]
    rate = (rand(n_reads) * 0.12 if e < 0 else
            torch.full((n_reads,), e / top, device=DEV) * (1.0 if cands == 1 else 2 * rand(n_reads)))

    letters = torch.tensor(_LETTERS, dtype=torch.uint8, device=DEV)
    text = []
    step = max(1, (1 << 26) // top)
    for a in range(0, n_reads, step):
        b = min(n_reads, a + step)
        u, r = rand(b - a, top), rate[a:b, None]
        sub, ins, dele = u < 0.7 * r, (u >= 0.7 * r) & (u < 0.85 * r), (u >= 0.85 * r) & (u < r)
        move = torch.ones_like(u, dtype=torch.int32)
        move[ins] = 0
        move[dele] = 2 + below(3, int(dele.sum())).int()
        idx = (origin[a:b, None] + torch.cumsum(move, 1, dtype=torch.int32) - 1).clamp(
            max=length - 1)
        col = torch.arange(top, device=DEV)[None]
        at = (rand(b - a) * (lens[a:b] - 12).clamp(min=1)).long()[:, None]
        seed_hit = ~true[a:b, None] & (col >= at) & (col < at + 12)
        idx = torch.where(seed_hit, (shared[a:b, None] + col).clamp(max=length - 1), idx)
        code = _bases(words, idx)
        change = below(3, b - a, top).int() + 1
        code = torch.where((sub | ins) & ~seed_hit, (code + change) & 3, code)
        chars = letters[code.long()]
        unknown = (rand(b - a) < 1 / 2000)[:, None] & (col == at)     # a base the caller left out
        chars[unknown] = 78
        text.append(chars[col < lens[a:b, None]] if m == 0 else chars.reshape(-1))
    off = torch.zeros(n_reads + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(lens, 0)
    return dict(n=n, n_reads=n_reads, top=top, text=torch.cat(text), off=off, lens=lens,
                pair_read=None if cands == 1 else pair_read.to(torch.int32),
                pos=pos.to(torch.int32), e=pair_e)


def _encoded(ctx, b):
    """The batch's reads as gk_encode_reads leaves them: (packed, lengths, unknown flags, pitch)."""
    rows, pitch = (b["top"] + 15) // 16, (b["n_reads"] + 63) // 64 * 64
    packed = torch.zeros(rows * pitch, dtype=torch.int32, device=DEV)
    lens = torch.zeros(b["n_reads"], dtype=torch.int16, device=DEV)
    has_n = torch.zeros(b["n_reads"], dtype=torch.uint8, device=DEV)
    return packed, lens, has_n, pitch


def _encode(ctx, b, out):
    packed, lens, has_n, pitch = out
    gk.gk_encode_reads(ctx, b["text"], b["off"], b["n_reads"], pitch, (b["top"] + 15) // 16,
                       gk.GK_READS_SPLIT, packed, lens, has_n)


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


_servers = {}


def _server(genome):
    if genome not in _servers:
        _servers[genome] = gk.gk_server_start(_genome(genome)[0], 2 << 30, 64, 512,
                                              gk.GK_SERVER_BATCHED)
    return _servers[genome]


def _burst(case, seed):
    """24 requests, sizes spread over a factor of 100 around the case's mean,
    each with one read length and one threshold."""
    r = np.random.default_rng(int(seed) + 5)
    size = np.geomspace(1, 100, 24)[np.arange(24) * 7 % 24]      # small and large ones in turn
    size = np.maximum(500, size / size.sum() * case["n"]).astype(int)
    reqs = []
    for k in range(24):
        m = int(r.integers(100, 251))
        one = dict(case, n=int(size[k]), m=m, e=int(r.integers(0, m // 10 + 1)))
        reqs.append((_batch(one, int(seed) * 64 + k), one["e"]))
    return reqs


def prepare(case, seed):
    ctx = _genome(case["genome"])[0]
    s = dict(case=case, ctx=ctx)
    if case["op"] == "served":
        s["server"] = _server(case["genome"])
        s["requests"] = []
        for b, e in _burst(case, seed):
            host = {k: _pinned(b[k]) for k in ("text", "off", "pos", "pair_read")}
            outs = [torch.zeros(b["n"], dtype=t, pin_memory=True)
                    for t in (torch.uint8, torch.int16)]
            s["requests"].append(gk.Request(
                host["text"].numpy(), host["off"].numpy().view(np.uint64),
                host["pos"].numpy().view(np.uint32), e,
                pair_read=host["pair_read"].numpy().view(np.uint32),
                accept=outs[0].numpy(), est=outs[1].numpy().view(np.uint16)))
            s.setdefault("keep", []).append((host, outs))
        return s
    b = _batch(case, seed)
    s["b"] = b
    if case["op"] == "host":
        for k in ("text", "off", "pos"):
            s[k] = _pinned(b[k])
        s["e"] = None if b["e"] is None else _pinned(b["e"])
        s["accept"] = torch.zeros(b["n"], dtype=torch.uint8, pin_memory=True)
        s["est"] = torch.zeros(b["n"], dtype=torch.int16, pin_memory=True)
        s["b"] = dict(n=b["n"], n_reads=b["n_reads"], top=b["top"])
        return s
    s["reads"] = _encoded(ctx, b)
    if case["op"] == "encode":
        return s
    if case["op"] != "ascii":
        _encode(ctx, b, s["reads"])
    n = b["n"]
    s["accept"] = torch.zeros(n, dtype=torch.uint8, device=DEV)
    s["est"] = torch.zeros(n, dtype=torch.int16, device=DEV)
    s["bits"] = torch.zeros((n + 63) // 64, dtype=torch.int64, device=DEV) if case["bits"] else None
    packed, lens, has_n, pitch = s["reads"]
    s["batch"] = gk.make_batch(
        n_reads=b["n_reads"], pitch=pitch, max_read_len=b["top"], reads=packed, read_len=lens,
        read_has_n=has_n, n_pairs=n, pair_read=b["pair_read"], cand_pos=b["pos"], e=b["e"],
        e_uniform=max(case["e"], 0), accept=s["accept"], est=s["est"], accept_bits=s["bits"])
    if case["op"] == "verify":
        gk.gk_filter(ctx, s["batch"])
        s["dist"] = torch.zeros(n, dtype=torch.int16, device=DEV)
    return s


def run(s):
    op, ctx = s["case"]["op"], s["ctx"]
    if op == "served":
        tickets = [gk.gk_server_submit(s["server"], q) for q in s["requests"]]
        for t in tickets:
            status, _ = gk.gk_server_wait(s["server"], t)
            if status != gk.GK_OK:
                raise gk.GkError(status, "gk_server_wait")
        return [(q.accept, q.est.view(np.int16)) for q in s["requests"]]
    b = s["b"]
    if op == "host":
        gk.gk_filter_host(ctx, s["text"], s["off"], s["pos"], s["accept"], s["est"],
                          max_read_len=b["top"], e=s["e"], e_uniform=max(s["case"]["e"], 0),
                          n_reads=b["n_reads"], n_pairs=b["n"])
    elif op == "encode":
        _encode(ctx, b, s["reads"])
        return s["reads"][:3]
    elif op == "filter":
        gk.gk_filter(ctx, s["batch"])
    elif op == "ascii":
        gk.gk_filter_ascii(ctx, s["batch"], b["text"], b["off"])
    elif op == "mixed":
        gk.gk_filter_mixed(ctx, s["batch"])
    elif op == "verify":
        gk.gk_verify(ctx, s["batch"], s["accept"], s["dist"])
        return s["dist"]
    return (s["accept"], s["est"]) + ((s["bits"],) if s.get("bits") is not None else ())


def work(case):
    """Bytes: reads, windows, pair entries and results, each once.  Flops:
    32-bit word operations, 4 for each 32 bases of a mask (compare two code
    bits, look for runs, collect), 12 for 32 cells of the edit-distance band."""
    n, m, e = case["n"], case["m"], case["e"]
    mean = (sum(MIX) / len(MIX) if case["op"] != "served" else 175.0) if m == 0 else m
    me = mean / 20 if e < 0 else e
    reads = n / case["cands"]
    if case["op"] == "encode":
        return {"bytes": n * (mean + 8 + mean / 4 + 3), "flops": 0.0}
    text = case["op"] in ("ascii", "host", "served")
    pair = 4 + (4 if case["cands"] > 1 else 0) + (1 if e < 0 else 0) + (0.125 if case["bits"] else 0)
    byts = reads * ((mean + 8) if text else (mean / 4 + 3)) + n * (pair + mean / 4)
    words = n * (2 * me + 1) * mean / 32
    if case["op"] == "verify":
        # about a third of the pairs were passed by the filter
        return {"bytes": byts / 3 + n * 3, "flops": 12.0 * words / 3}
    return {"bytes": byts + n * 3, "flops": 4.0 * words}


# ------------------------------------------------------------------- exact ---

def _opened(match):
    """Runs of three or more matches; a run that touches an end counts whole."""
    z = torch.nn.functional.pad(match, (2, 2), value=True)
    three = z[:, :-2] & z[:, 1:-1] & z[:, 2:]
    return three[:, :-2] | three[:, 1:-1] | three[:, 2:]


def _masks(read, window, e, m):
    """Edit estimates of reads of one length m (codes) under thresholds e."""
    n = read.shape[0]
    found = _opened(read == window)
    for k in range(1, min(int(e.max()), m - 1) + 1):
        on = (e >= k)[:, None]
        zero = torch.zeros((n, k), dtype=read.dtype, device=DEV)
        d = _opened(torch.cat([zero, read[:, :-k]], 1) == window)
        i = _opened(torch.cat([read[:, k:], zero], 1) == window)
        d[:, :k] = False
        i[:, m - k:] = False
        found |= (d | i) & on
    return m - found.sum(1)


def _distance(read, window, e, m):
    """min(edit distance, e + 1), row by row of the whole matrix."""
    n = read.shape[0]
    j = torch.arange(m + 1, device=DEV, dtype=torch.int32)
    row = j.expand(n, m + 1)
    for i in range(1, m + 1):
        t = torch.empty_like(row)
        t[:, 0] = i
        t[:, 1:] = torch.minimum(row[:, :-1] + (read[:, i - 1:i] != window), row[:, 1:] + 1)
        row = torch.cummin(t - j, 1).values + j
    return torch.minimum(row[:, m], e + 1)


def exact(case, seed):
    """Codes, estimates and distances from plain tensor operations on each
    base, for the cases small enough."""
    _, length, words, runs = _genome(case["genome"])
    if case["op"] in ("served", "encode") or work(case)["flops"] > 2e9:
        return None
    if case["op"] == "verify" and case["n"] * (case["m"] or 200) ** 2 > 4e10:
        return None
    b = _batch(case, seed)
    n = b["n"]
    pr = torch.arange(n, device=DEV) if b["pair_read"] is None else b["pair_read"].long()
    pos = b["pos"].long() & 0xFFFFFFFF
    lens = b["lens"][pr]
    e = torch.full((n,), case["e"], device=DEV) if b["e"] is None else b["e"].long()
    accept = torch.zeros(n, dtype=torch.uint8, device=DEV)
    est = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    dist = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    for m in sorted(set(lens.tolist())):
        rows = torch.nonzero(lens == m)[:, 0]
        for part in rows.split(max(1, (1 << 26) // m)):
            col = torch.arange(m, device=DEV)[None]
            chars = b["text"][b["off"][pr[part]][:, None] + col]
            idx = pos[part][:, None] + col
            unknown = (chars == 78).any(1)
            for at, size in (() if runs is None else runs.astype(np.int64)):
                unknown |= (pos[part] < int(at + size)) & (pos[part] + m > int(at))
            read = ((chars >> 1) ^ (chars >> 2)) & 3
            window = _bases(words, idx).to(torch.uint8)
            c = _masks(read, window, e[part], m)
            ok = (c <= e[part]).to(torch.uint8)
            accept[part] = torch.where(unknown, torch.full_like(ok, 2), ok)
            est[part] = torch.where(unknown, -1, c).to(torch.int16)
            if case["op"] == "verify":
                sub = (accept[part] == 1) & (e[part] <= gk.GK_VERIFY_MAX_E)
                keep = part[sub]
                if keep.numel():
                    dist[keep] = _distance(read[sub], window[sub], e[keep].int(), m).to(torch.int16)
    if case["op"] == "verify":
        return dist
    if case["op"] == "host":
        return accept.cpu(), est.cpu()
    if not case["bits"]:
        return accept, est
    on = torch.nn.functional.pad(((accept == 1) | (accept == 2)).long(), (0, -n % 64))
    return accept, est, (on.reshape(-1, 64) << torch.arange(64, device=DEV)).sum(1)
