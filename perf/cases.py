"""Performance cases of the SNP-profile comparison: the work that a program using this package has it do, through
its public entry points, from one small count matrix to a whole ragged batch.

Profiles are synthetic, made on the GPU from the seed alone with the recipe of gen/workloads.py (per-locus minor-allele
frequency uniform in [lo, 0.5), mixtures of 1-4 database references with 0.5% flipped bits, identity queries one
reference with the same flips), but drawn with torch as packed words, which takes milliseconds.

The operations, by the case's "op":
  topk       Context.compare_topk: the k nearest references of each query (compare_topk_mixed with mode "mixed")
  full       Context.compare_full: the whole count matrix
  tiles      Context.compare_tiles: blocks of the matrix at arbitrary origins
  threshold  Context.compare_threshold: every reference within a count of 2% of the loci
  both       Context.compare_threshold_topk: the two reports of a search from one pass
  ingest     Context.pack or pack_genotypes, build_db, popcounts: locus bytes to a searchable database
  streamed   Context.compare_topk_streamed: the database stays in pinned host memory
  batch      fid_batch_run: independent top-k jobs over slices of resident panels
  serve      Server.submit and wait: a burst of requests against one resident database
"""
import math
import random

import torch

import paper_1707_00516_amd as fid
from paper_1707_00516_amd import autotune
from paper_1707_00516_amd.torch_api import Context, Server, row_words

MIXTURE, IDENTITY = fid.FID_MODE_MIXTURE, fid.FID_MODE_IDENTITY
PANELS = (1024, 2048, 4096, 8192, 16384)   # loci panels of the ragged batches


def listed():
    return [
        # one evidence batch against a local database, every count wanted: the smallest call, all launch latency
        dict(name="full-64x20k-2048", op="full", mode="mixture", n_q=64, n_refs=20_000, n_loci=2048),
        # one profile looked up in a national database: reads the database once
        dict(name="lookup-1x20M-2048", op="topk", mode="identity", n_q=1, n_refs=20_000_000, n_loci=2048, k=32),
        # one tick of a serving loop: 131 waiting queries of both modes, as many as the served load holds on average
        dict(name="tick-131x20M-2048", op="topk", mode="mixed", n_q=131, n_refs=20_000_000, n_loci=2048, k=32),
        # the headline search: 2,048 unknown mixtures against 20 million known profiles
        dict(name="search-2048x20M-2048", op="topk", mode="mixture", n_q=2048, n_refs=20_000_000, n_loci=2048, k=32),
        # the short SNP panels of the paper (up to 512 SNPs), 512 unknowns, a database of 10 million
        dict(name="panel512-512x10M", op="topk", mode="mixture", n_q=512, n_refs=10_000_000, n_loci=512, k=32),
        # the paper's own output: the whole count matrix, 8.2 GB of it
        dict(name="full-2048x1M-2048", op="full", mode="mixture", n_q=2048, n_refs=1_000_000, n_loci=2048),
        # dense genotyping chips: 32,768 loci, all references within 2% and the nearest 32 from one pass
        dict(name="chip-256x2M-32768", op="both", mode="mixture", n_q=256, n_refs=2_000_000, n_loci=32768, k=32),
        # kinship screening on a panel of no round length: every reference within 2% of an individual
        dict(name="screen-300x1M-1000", op="threshold", mode="identity", n_q=300, n_refs=1_000_000, n_loci=1000),
        # a laboratory's job list: 400 searches of ragged sizes over five panels in one run
        dict(name="ragged-400", op="batch", jobs=400, pool=2_000_000, k=32, graph=False),
        # loading a database: 0/1 locus bytes to packed rows to the resident form
        dict(name="ingest-500k-2048", op="ingest", geno=False, n_refs=500_000, n_loci=2048),
        # a database too large to keep resident passes through from host memory
        dict(name="streamed-128x1M-2048", op="streamed", mode="mixture", n_q=128, n_refs=1_000_000, n_loci=2048, k=32,
             block=131_072),
        # eight requests of 1-256 queries arrive at once, two of them asking for threshold hits as well
        dict(name="serve-8x20M-2048", op="serve", requests=8, n_refs=20_000_000, n_loci=2048, k=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(("topk", "topk", "topk", "full", "full", "threshold", "both", "ingest", "batch", "serve", "tiles",
                     "streamed"))
    n_loci = _log(rng, 96, 16384) if rng.random() < 0.6 else rng.choice((128, 256, 512) + PANELS)
    mode = rng.choice(("mixture", "identity"))
    if op == "topk":
        # up to the listed sizes; at most 8 GB of packed profiles
        n_refs = _log(rng, 5_000, min(20_000_000, 64_000_000_000 // n_loci))
        return dict(op=op, mode=rng.choice((mode, mode, "mixed")), n_q=_log(rng, 1, 2048), n_refs=n_refs,
                    n_loci=n_loci, k=rng.choice((1, 10, 32, 32, 100)))
    if op == "full":
        n_q = _log(rng, 1, 2048)
        return dict(op=op, mode=mode, n_q=n_q, n_refs=_log(rng, 2_000, min(1_000_000, 1_000_000_000 // n_q)),
                    n_loci=n_loci)
    if op in ("threshold", "both"):
        # on fewer loci 2% no longer separates the contributors from strangers
        n_loci = max(n_loci, 512 if mode == "identity" else 2048)
        c = dict(op=op, mode=mode, n_q=_log(rng, 8, 512), n_refs=_log(rng, 20_000, 2_000_000), n_loci=n_loci)
        return dict(c, k=rng.choice((10, 32))) if op == "both" else c
    if op == "ingest":
        geno = rng.random() < 0.5
        n_loci = min(n_loci, 8192)
        return dict(op=op, geno=geno, n_refs=_log(rng, 1_000, min(1_000_000, 1_500_000_000 // n_loci)), n_loci=n_loci)
    if op == "batch":
        return dict(op=op, jobs=rng.randint(3, 60), pool=_log(rng, 50_000, 1_000_000), k=rng.choice((10, 32)),
                    graph=rng.random() < 0.5)
    if op == "serve":
        return dict(op=op, requests=rng.randint(1, 12), n_refs=_log(rng, 100_000, 5_000_000),
                    n_loci=min(n_loci, 4096), k=rng.choice((10, 32)))
    if op == "tiles":
        return dict(op=op, mode=mode, tiles=rng.randint(1, 64), side=rng.choice((32, 100, 256)), n_q=_log(rng, 256, 2048),
                    n_refs=_log(rng, 20_000, 500_000), n_loci=n_loci)
    n_refs = _log(rng, 50_000, min(1_000_000, 2_000_000_000 // n_loci))
    return dict(op=op, mode=mode, n_q=_log(rng, 1, 512), n_refs=n_refs, n_loci=n_loci, k=rng.choice((10, 32)),
                block=max(4096, n_refs // rng.randint(2, 9)))


# ------------------------------------------------------------------------------------------------------- inputs
def _gen(case, seed):
    return torch.Generator(device="cuda").manual_seed(seed * 1_000_003 + sum(map(ord, case["op"])))


def _bernoulli(g, prob, n, n_loci, bits):
    """n packed rows whose locus k is set with probability prob[k] / 2**bits (prob: int64 [n_loci])."""
    rw = row_words(n_loci)
    # bit b of every locus's probability, as packed words
    pad = torch.zeros(rw * 64, dtype=torch.int64, device="cuda")
    pad[:n_loci] = prob
    place = torch.arange(64, device="cuda")
    masks = [(((pad >> b) & 1).view(rw, 64) << place).sum(1) for b in range(bits)]
    live = ((pad > 0).to(torch.int64).view(rw, 64) << place).sum(1)
    out = torch.empty((n, rw), dtype=torch.int64, device="cuda")
    step = max(1, (1 << 25) // rw)
    for i in range(0, n, step):
        x = out[i:i + step].zero_()
        r = torch.empty_like(x)
        for b in range(bits):  # P(x) <- (bit b + P(x)) / 2
            r.random_(-(1 << 63), None, generator=g)
            x.copy_((r & x) | (masks[b] & (r | x)))
        x &= live
    return out


def _rows(g, n, n_loci):
    lo = 0.01 if n_loci >= 32768 else 0.05
    maf = lo + (0.5 - lo) * torch.rand(n_loci, dtype=torch.float64, device="cuda", generator=g)
    return _bernoulli(g, (maf * 256).long().clamp_(1, 255), n, n_loci, 8)


def _queries(g, rows, n_loci, modes, lo=0, n=None):
    """One query per entry of modes (0 mixture of 1-4 rows, 1 one row) from rows [lo, lo + n), with flipped bits;
    lo and n may be tensors with one entry per query."""
    n_q = modes.numel()
    n = torch.full_like(modes, rows.shape[0], dtype=torch.int64) if n is None else n
    u = torch.rand((n_q, 2), dtype=torch.float64, device="cuda", generator=g)
    first, step = (u[:, 0] * n).long(), 1 + (u[:, 1] * (n // 4 - 1)).long()   # four distinct rows
    count = torch.where(modes == IDENTITY, 1, 1 + torch.arange(n_q, device="cuda") % 4)
    q = rows[lo + first]
    for j in range(1, 4):
        q = torch.where((count > j)[:, None], q | rows[lo + (first + j * step) % n], q)
    flip = _bernoulli(g, torch.full((n_loci,), 328, dtype=torch.int64, device="cuda"), n_q, n_loci, 16)
    return (q ^ flip).contiguous()


def _modes(case, g, n_q):
    if case.get("mode") == "mixed":
        return torch.randint(0, 2, (n_q,), device="cuda", generator=g, dtype=torch.int32)
    return torch.full((n_q,), IDENTITY if case.get("mode") == "identity" else MIXTURE, dtype=torch.int32, device="cuda")


def _search_inputs(case, seed):
    g = _gen(case, seed)
    rows = _rows(g, case["n_refs"], case["n_loci"])
    modes = _modes(case, g, case["n_q"])
    return rows, _queries(g, rows, case["n_loci"], modes), modes


def _tile_origins(case):
    r = random.Random(case["tiles"])
    s = case["side"]
    return [(r.randint(0, case["n_q"] - s), r.randint(0, case["n_refs"] - s)) for _ in range(case["tiles"])]


def _ingest_bytes(case, seed):
    g = _gen(case, seed)
    n, n_loci = case["n_refs"], case["n_loci"]
    maf = 0.05 + 0.45 * torch.rand(n_loci, device="cuda", generator=g)
    data = torch.empty((n, n_loci), dtype=torch.uint8, device="cuda")
    for i in range(0, n, max(1, (1 << 26) // n_loci)):
        x = data[i:i + max(1, (1 << 26) // n_loci)]
        for _ in range(2 if case["geno"] else 1):
            hit = torch.rand(x.shape, device="cuda", generator=g) < maf
            x.copy_(x + hit if _ else hit)
    return data


def _job_table(case):
    """(n_q, r_lo, n_refs, loci, mode) of every job: sizes are the case's own, not the seed's."""
    r = random.Random(case["jobs"] * 7 + 3)
    pool = case["pool"]
    table = []
    for _ in range(case["jobs"]):
        n = r.randint(min(10_000, pool), pool)
        table.append((r.randint(1, 512), r.randint(0, pool - n), n, r.choice(PANELS), r.randint(0, 1)))
    return table


def _request_table(case):
    """(queries, mode, wants threshold hits) of every request."""
    r = random.Random(case["requests"] * 11 + 5)
    table = [(r.randint(1, 256), r.randint(0, 1)) for _ in range(case["requests"])]
    return [(n_q, mode, i % 4 == 3 and case["n_loci"] >= (512 if mode == IDENTITY else 2048))
            for i, (n_q, mode) in enumerate(table)]


def _batch_inputs(case, seed):
    g = _gen(case, seed)
    table = _job_table(case)
    pools, queries = {}, [None] * len(table)
    for n_loci in sorted({t[3] for t in table}):
        rows = pools[n_loci] = _rows(g, case["pool"], n_loci)
        mine = [(j, t) for j, t in enumerate(table) if t[3] == n_loci]
        each = [torch.full((t[0],), v, dtype=torch.int64, device="cuda") for _, t in mine for v in (t[4], t[1], t[2])]
        q = _queries(g, rows, n_loci, torch.cat(each[0::3]), torch.cat(each[1::3]), torch.cat(each[2::3]))
        for (j, _), part in zip(mine, q.split([t[0] for _, t in mine])):
            queries[j] = part
    return table, pools, queries


# ------------------------------------------------------------------------------------------------------- cases
def prepare(case, seed):
    op = case["op"]
    ctx = Context(0)
    if op == "ingest":
        return dict(case=case, ctx=ctx, data=_ingest_bytes(case, seed))
    if op == "batch":
        table, pools, queries = _batch_inputs(case, seed)
        dbs = {n: ctx.build_db(rows, n) for n, rows in pools.items()}
        ctx.sync()
        total, k = sum(t[0] for t in table), case["k"]
        cnt = torch.empty((total, k), dtype=torch.int32, device="cuda")
        idx = torch.empty((total, k), dtype=torch.int64, device="cuda")
        jobs, at, tune = [], 0, autotune.load_table()
        for (n_q, lo, n, n_loci, mode), q in zip(table, queries):
            jobs.append(fid.FidJob(dbs[n_loci].handle, lo, lo + n, q.data_ptr(), n_q, mode, cnt[at:].data_ptr(),
                                   idx[at:].data_ptr()))
            at += n_q
        ws = torch.empty(max(16, fid.fid_batch_workspace_bytes(ctx.handle, jobs, k, tune)), dtype=torch.uint8,
                         device="cuda")
        plan = _Plan(fid.fid_batch_create(ctx.handle, jobs, k, tune, ws.data_ptr(), ws.numel()))
        return dict(case=case, plan=plan, out=(cnt, idx), ws=ws, queries=queries, dbs=dbs, ctx=ctx)
    if op == "serve":
        g = _gen(case, seed)
        rows = _rows(g, case["n_refs"], case["n_loci"])
        table = _request_table(case)
        queries = [_queries(g, rows, case["n_loci"], torch.full((n_q,), mode, device="cuda"))
                   for n_q, mode, _ in table]
        db = ctx.build_db(rows, case["n_loci"])
        ctx.sync()
        server = Server(ctx, db, 16 << 30, 4096, case["k"], 8, fid.FID_SERVE_CONTINUOUS, 0, 16)
        return dict(case=case, server=server, table=table, queries=queries, db=db, ctx=ctx)
    rows, q, modes = _search_inputs(case, seed)
    n_q, n_refs = case["n_q"], case["n_refs"]
    mode = IDENTITY if case["mode"] == "identity" else MIXTURE
    state = dict(case=case, ctx=ctx, q=q, mode=mode)
    if op == "streamed":
        host = torch.empty(rows.shape, dtype=torch.int64, pin_memory=True)
        host.copy_(rows)
        need = fid.fid_stream_workspace_bytes(ctx.handle, n_refs, case["n_loci"], case["block"], n_q, case["k"])
        return dict(state, host=host, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
    db = state["db"] = ctx.build_db(rows, case["n_loci"])
    ctx.sync()
    if op == "topk":
        if case["mode"] == "mixed":
            need = fid.fid_topk_mixed_workspace_bytes(ctx.handle, db.handle, 0, n_refs, n_q, case["k"])
            state.update(modes=modes, ws=torch.empty(max(16, need), dtype=torch.uint8, device="cuda"))
        else:
            state["ws"] = ctx.topk_workspace(db, n_q, case["k"])
    elif op == "full":
        state["out"] = torch.empty((n_q, n_refs), dtype=torch.int32, device="cuda")
    elif op == "tiles":
        state["origins"] = _tile_origins(case)
    elif op in ("threshold", "both"):
        state["thr"] = torch.full((n_q,), 2 * case["n_loci"] // 100, dtype=torch.int32, device="cuda")
    return state


class _Plan:
    """A batch handle that is given back with its state."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        try:
            fid.fid_batch_destroy(self.handle)
        except Exception:
            pass


def run(state):
    case = state["case"]
    op, ctx = case["op"], state["ctx"]
    if op == "topk":
        if case["mode"] == "mixed":
            return ctx.compare_topk_mixed(state["db"], 0, case["n_refs"], state["q"], state["modes"], case["k"],
                                          ws=state["ws"])
        return ctx.compare_topk(state["db"], state["q"], state["mode"], case["k"], ws=state["ws"])
    if op == "full":
        return ctx.compare_full(state["db"], state["q"], state["mode"], out=state["out"])
    if op == "tiles":
        return ctx.compare_tiles(state["db"], state["q"], state["mode"], state["origins"], case["side"], case["side"])
    if op == "threshold":
        return ctx.compare_threshold(state["db"], state["q"], state["mode"], state["thr"])
    if op == "both":
        return ctx.compare_threshold_topk(state["db"], state["q"], state["mode"], state["thr"], case["k"])
    if op == "ingest":
        n_loci = case["n_loci"]
        if case["geno"]:
            rows, n_loci = ctx.pack_genotypes(state["data"]), 2 * n_loci
        else:
            rows = ctx.pack(state["data"])
        db = ctx.build_db(rows, n_loci)
        return rows, db.popcounts()
    if op == "streamed":
        return ctx.compare_topk_streamed(state["host"], case["n_loci"], case["block"], state["q"], state["mode"],
                                         case["k"], ws=state["ws"])
    if op == "batch":
        fid.fid_batch_run(state["plan"].handle, case["graph"])
        return state["out"]
    server, thr = state["server"], 2 * case["n_loci"] // 100
    tickets = [server.submit(q, mode, thr=thr if hits else None)
               for q, (_, mode, hits) in zip(state["queries"], state["table"])]
    done = [server.wait(t) for t in tickets]
    return [(r[0], r[1]) + tuple(r[3:]) for r in done]


def work(case):
    """Packed profiles, queries and locus bytes read once, outputs written once; a comparison of one locus is one
    multiply-add."""
    op = case["op"]
    if op == "ingest":
        n, n_loci = case["n_refs"], case["n_loci"]
        rows = 8 * row_words(2 * n_loci if case["geno"] else n_loci) * n
        return {"bytes": n * n_loci + 2 * rows + 4 * n, "flops": 0}
    if op == "batch":
        table, k = _job_table(case), case["k"]
        read = {}
        for n_q, lo, n, n_loci, _ in table:  # each panel's rows that any job covers, once
            read.setdefault(n_loci, []).append((lo, lo + n))
        nbytes = 0
        for n_loci, spans in read.items():
            end = 0
            for a, b in sorted(spans):
                nbytes += max(0, b - max(a, end)) * 8 * row_words(n_loci)
                end = max(end, b)
        return {"bytes": nbytes + sum(t[0] * (8 * row_words(t[3]) + 12 * k) for t in table),
                "flops": 2 * sum(t[0] * t[2] * t[3] for t in table)}
    n_refs, n_loci = case["n_refs"], case["n_loci"]
    row = 8 * row_words(n_loci)
    if op == "serve":
        n_q = sum(t[0] for t in _request_table(case))
        return {"bytes": n_refs * row + n_q * (row + 12 * case["k"]), "flops": 2 * n_q * n_refs * n_loci}
    n_q = case["n_q"]
    if op == "tiles":
        at, s = _tile_origins(case), case["side"]
        return {"bytes": len(at) * (2 * s * row + 4 * s * s), "flops": 2 * len(at) * s * s * n_loci}
    out = 4 * n_q * n_refs if op == "full" else 12 * n_q * case.get("k", 1)
    return {"bytes": n_refs * row + n_q * row + out, "flops": 2 * n_q * n_refs * n_loci}


# ------------------------------------------------------------------------------------------------------- exact values
def _unpack(rows, n_loci):
    """Packed rows [n, row_words] -> 0.0/1.0 float64 [n, n_loci]."""
    b = (rows[:, :, None] >> torch.arange(64, device=rows.device)) & 1
    return b.view(rows.shape[0], -1)[:, :n_loci].double()


def _counts(rows, q, modes, n_loci):
    """Exact counts [n_q, n] of packed rows in 64-bit arithmetic."""
    r, x = _unpack(rows, n_loci), _unpack(q, n_loci)
    dot, pr, pq = x @ r.T, r.sum(1)[None, :], x.sum(1)[:, None]
    ident = (modes == IDENTITY)[:, None]
    return torch.where(ident, pr + pq - 2 * dot, pr - dot).long()


def _exact_search(rows, q, modes, n_loci, lo=0, k=None, thr=None):
    """Top-k (cnt, idx) and threshold hits (offs, idx, cnt) over rows, references numbered from lo."""
    best, hits = None, []
    step = max(1, min((1 << 27) // max(q.shape[0], 1), (1 << 26) // n_loci))
    for i in range(0, rows.shape[0], step):
        c = _counts(rows[i:i + step], q, modes, n_loci)
        at = torch.arange(lo + i, lo + i + c.shape[1], device="cuda")
        if k:
            key = (c << 40) | at
            key = key if best is None else torch.cat((best, key), 1)
            best = key.topk(min(k, key.shape[1]), dim=1, largest=False, sorted=True).values
        if thr is not None:
            w = (c <= thr).nonzero()
            hits.append((w[:, 0], at[w[:, 1]], c[w[:, 0], w[:, 1]]))
    got = []
    if thr is not None:
        who, at, c = (torch.cat(x) for x in zip(*hits))
        order = (who * (1 << 40) + at).argsort()
        offs = torch.cat((torch.zeros(1, dtype=torch.int64, device="cuda"),
                          torch.bincount(who, minlength=q.shape[0]).cumsum(0)))
        got += [offs, at[order], c[order].int()]
    if k:
        short = k - best.shape[1]
        cnt, idx = (best >> 40).int(), best & ((1 << 40) - 1)
        if short:
            cnt = torch.cat((cnt, torch.full((q.shape[0], short), 2**31 - 1, dtype=torch.int32, device="cuda")), 1)
            idx = torch.cat((idx, torch.full((q.shape[0], short), -1, dtype=torch.int64, device="cuda")), 1)
        got += [cnt, idx]
    return tuple(got)


def exact(case, seed):
    """What run() returns, from 64-bit matrix products and sorts in torch; None where that takes too long."""
    w = work(case)
    if w["flops"] > 2e13 or w["bytes"] > 6e9:
        return None
    op = case["op"]
    if op == "ingest":
        data = _ingest_bytes(case, seed)
        if case["geno"]:
            data = torch.stack((data >= 1, data >= 2), 2).view(data.shape[0], -1)
        rw = row_words(data.shape[1])
        out = torch.empty((data.shape[0], rw), dtype=torch.int64, device="cuda")
        step = max(1, (1 << 25) // (rw * 64))
        for i in range(0, data.shape[0], step):
            x = torch.zeros((min(step, data.shape[0] - i), rw * 64), dtype=torch.int64, device="cuda")
            x[:, :data.shape[1]] = data[i:i + step]
            out[i:i + step] = (x.view(-1, rw, 64) << torch.arange(64, device="cuda")).sum(2)
        return out, data.sum(1, dtype=torch.int32)
    if op == "batch":
        table, pools, queries = _batch_inputs(case, seed)
        done = [_exact_search(pools[n_loci][lo:lo + n], q, torch.full((n_q,), mode, device="cuda"), n_loci, lo,
                              case["k"])
                for (n_q, lo, n, n_loci, mode), q in zip(table, queries)]
        return tuple(torch.cat(x) for x in zip(*done))
    n_loci = case["n_loci"]
    thr = 2 * n_loci // 100
    if op == "serve":
        g = _gen(case, seed)
        rows = _rows(g, case["n_refs"], n_loci)
        done = []
        for n_q, mode, hits in _request_table(case):
            modes = torch.full((n_q,), mode, device="cuda")
            got = _exact_search(rows, _queries(g, rows, n_loci, modes), modes, n_loci, 0, case["k"],
                                thr if hits else None)
            done.append(tuple(got[-2:]) + ((tuple(got[:3]),) if hits else ()))
        return done
    rows, q, modes = _search_inputs(case, seed)
    if op == "full":
        step = max(1, (1 << 26) // n_loci)
        return torch.cat([_counts(rows[i:i + step], q, modes, n_loci).int()
                          for i in range(0, rows.shape[0], step)], 1)
    if op == "tiles":
        s = case["side"]
        return torch.stack([_counts(rows[r0:r0 + s], q[q0:q0 + s], modes[q0:q0 + s], n_loci).int()
                            for q0, r0 in _tile_origins(case)])
    return _exact_search(rows, q, modes, n_loci, 0, case.get("k"), thr if op in ("threshold", "both") else None)
