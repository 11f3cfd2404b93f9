"""Timed cases of the library, through its public entry points: what a memory
service does with it, from one user's question to the 1M-chunk batch, over
both embedding types, every list length and ragged sizes.

Kinds of case:

* ``retrieve``  -- mem_retrieve_topk: queries against a resident bank.
* ``step``      -- retrieval, then mem_gather_chunks of the selected blocks in
  time order (the benchmark's step).
* ``round``     -- one streaming round: the new chunks' related chunks, then
  mem_append_chunks.
* ``relations`` -- mem_build_relations over a whole bank.
* ``scoped``    -- mem_retrieve_topk_scoped: one bank for all (user, session)
  namespaces, some rows tombstoned.
* ``request``   -- mem_retrieve_topk_grouped over the chunk tables, then the
  prompt prefix of mem_gather_budget.
* ``maintain``  -- mem_colocate of strongly related chunks, then
  mem_compact_blocks of the blocks that hold the stale copies.

Embeddings are the Gaussian mixture of ``inputs.py`` (centroid + 0.3 noise,
L2-normalised; a query is a perturbed member), drawn on the GPU.
"""
import math

import torch

import paper_2607_05708_amd as pm

DEV = "cuda"
BLOCK = 65536  # bank rows drawn at a time


def listed():
    return [
        # the smallest call in the tests and the benchmark: fp32 embeddings, every probability wanted
        dict(name="tiny_fp32_probs", kind="retrieve", dtype="f32", m=16, n=1024, d=256, k=8, probs=True),
        # one user's question against a few thousand memories, the paper's default of 5 chunks
        dict(name="one_query", kind="retrieve", dtype="bf16", m=1, n=4096, d=1024, k=5, probs=False),
        # an embedder that gives fp32: a batch of questions against a medium bank
        dict(name="fp32_batch", kind="retrieve", dtype="f32", m=64, n=65536, d=768, k=16, probs=False),
        # short fp32 vectors of a dimension no tile divides, ragged bank
        dict(name="fp32_ragged", kind="retrieve", dtype="f32", m=33, n=70001, d=100, k=24, probs=False),
        # the longest lists the library returns (a reranker's input), ragged bank and batch
        dict(name="bf16_top64", kind="retrieve", dtype="bf16", m=200, n=100003, d=1024, k=64, probs=False),
        # the benchmark's batched retrieval
        dict(name="batched_262k", kind="retrieve", dtype="bf16", m=512, n=262144, d=1024, k=16, probs=False),
        # the benchmark's step: 1,024 queries, 1M chunks, top-32, 4 GiB of blocks in time order
        dict(name="step_1M", kind="step", m=1024, n=1048576, d=1024, k=32, ppc=2, page=65536, pages=65536),
        # a small streaming round against the 1M bank
        dict(name="round_1M_m16", kind="round", m=16, n=1048576, d=1024, k=32, ppc=2),
        # the benchmark's relation build
        dict(name="relations_32k", kind="relations", n=32768, d=768, k=32),
        # a shared 1M bank of 256 namespaces, sessions appending in bursts of 64 rows, 10 % tombstones
        dict(name="scoped_1M", kind="scoped", m=1024, n=1048576, d=1024, k=32, spaces=256, burst=64),
        # the paper's request path: top-5 of each request's own table, then the prefix within 1,536 tokens
        dict(name="request_1M", kind="request", m=1024, n=1048576, d=1024, k=5, spaces=256, burst=64, budget=1536,
             ppc=2, page=65536, pages=65536),
        # the background stage over 4 GiB of written blocks of 4 MiB
        dict(name="maintain_4GiB", kind="maintain", blocks=1024, per_block=64, page=65536, ppc=2, m=256, k=32,
             spaces=64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["retrieve", "retrieve", "retrieve", "retrieve", "step", "round", "relations", "scoped",
                       "request", "maintain"])
    dims = [64, 96, 128, 256, 384, 512, 768, 1024]
    if kind == "retrieve":
        dtype = rng.choice(["f32", "bf16", "bf16"])
        d = rng.choice([20, 100, 200, 300] + dims) if rng.random() < 0.8 else rng.randint(16, 1024)
        k = rng.randint(1, 64)
        m, n = _log(rng, 1, 1024), _log(rng, 1000, 1 << 20)
        # a call that the matrix-core path cannot take costs no more than bf16_top64, any other no more than step_1M
        most = 1024 << 30 if dtype == "bf16" and d % 32 == 0 and k <= 32 else 200 * 100003 * 1024
        while m * n * d > most:
            m, n = max(1, m * 2 // 3), max(1000, n * 2 // 3)
        probs = rng.random() < 0.25 and m * n <= 1 << 22
        return dict(kind=kind, dtype=dtype, m=m, n=n, d=d, k=k, probs=probs)
    if kind == "step":
        m = _log(rng, 16, 1024)
        return dict(kind=kind, m=m, n=_log(rng, 20000, 1 << 20), d=rng.choice(dims), k=rng.randint(1, 32),
                    ppc=rng.choice([1, 2, 3]), page=rng.choice([4096, 16384, 32768]), pages=65536)
    if kind == "round":
        return dict(kind=kind, m=_log(rng, 1, 1024), n=_log(rng, 20000, 1 << 20), d=rng.choice(dims),
                    k=rng.randint(1, 32), ppc=rng.choice([1, 2, 4]))
    if kind == "relations":
        return dict(kind=kind, n=_log(rng, 2000, 32768), d=rng.choice(dims[:7]), k=rng.randint(1, 32))
    if kind == "scoped":
        return dict(kind=kind, m=_log(rng, 16, 1024), n=_log(rng, 20000, 1 << 20), d=rng.choice(dims),
                    k=rng.randint(1, 32), spaces=_log(rng, 8, 1024), burst=rng.choice([1, 16, 64]))
    if kind == "request":
        return dict(kind=kind, m=_log(rng, 16, 1024), n=_log(rng, 20000, 1 << 20), d=rng.choice(dims[1:]),
                    k=rng.randint(1, 32), spaces=_log(rng, 8, 1024), burst=rng.choice([1, 16, 64]),
                    budget=rng.choice([512, 1000, 1536, 3072]), ppc=2, page=65536, pages=32768)
    return dict(kind=kind, blocks=_log(rng, 64, 1024), per_block=rng.choice([16, 64]), page=rng.choice([16384, 65536]),
                ppc=rng.choice([1, 2, 4]), m=_log(rng, 16, 256), k=rng.randint(4, 32), spaces=_log(rng, 4, 256))


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _mixture(g, n, d, m, dtype, extra=0):
    """(bank [n + extra, d] with n rows drawn, m queries, each query's source row): clusters of about 1,024 rows at
    1M rows and 128 at 32,768."""
    clusters = max(4, min(1024, n // 128))
    cent = torch.randn((clusters, d), generator=g, device=DEV)
    bank = torch.zeros((n + extra, d), dtype=dtype, device=DEV)
    src = torch.randint(0, n, (m,), generator=g, device=DEV)
    raw_q = torch.zeros((m, d), device=DEV)
    for r0 in range(0, n, BLOCK):
        r1 = min(n, r0 + BLOCK)
        c = torch.randint(0, clusters, (r1 - r0,), generator=g, device=DEV)
        raw = cent[c] + 0.3 * torch.randn((r1 - r0, d), generator=g, device=DEV)
        bank[r0:r1] = torch.nn.functional.normalize(raw, dim=1).to(dtype)
        here = ((src >= r0) & (src < r1))[:, None]
        raw_q = torch.where(here, raw[(src - r0).clamp(0, r1 - r0 - 1)], raw_q)
    raw_q += 0.2 * torch.randn((m, d), generator=g, device=DEV)
    return bank, torch.nn.functional.normalize(raw_q, dim=1).to(dtype), src


def _namespaces(g, n, spaces, burst, dead=0.1):
    """Namespace per row in bursts of about `burst` rows, -1 for a tombstoned row."""
    run = (torch.rand(n, generator=g, device=DEV) < 1.0 / burst).to(torch.int64).cumsum(0)
    ns = torch.randint(0, spaces, (n + 1,), generator=g, device=DEV)[run]
    live = torch.rand(n, generator=g, device=DEV) >= dead
    return ns.to(torch.int32), torch.where(live, ns, -1).to(torch.int32)


def _tables(row_ns, spaces):
    """CSR chunk tables of the live rows."""
    live = torch.nonzero(row_ns >= 0).flatten()
    order = live[torch.sort(row_ns[live], stable=True).indices]
    counts = torch.bincount(row_ns[live].to(torch.int64), minlength=spaces)
    offsets = torch.cat([counts.new_zeros(1), counts.cumsum(0)])
    return offsets.to(torch.int32), order.to(torch.int32)


def _pool(g, pages, page):
    return torch.empty((pages, page // 8), dtype=torch.int64, device=DEV).random_(generator=g)


def _directory(g, n, ppc, pages):
    """Page table over a pool that holds fewer chunks than the bank (their payload is not what is timed)."""
    return torch.randint(0, pages, (n, ppc), generator=g, device=DEV, dtype=torch.int32)


def _out(m, k):
    return (torch.empty((m, k), dtype=torch.int32, device=DEV), torch.empty((m, k), device=DEV),
            torch.empty((m, k), device=DEV), torch.empty((m,), device=DEV))


def _bytes(nbytes):
    return torch.empty(max(1, nbytes), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case)
    if kind == "maintain":
        return _prepare_maintain(s, g)
    m, n, d, k = case.get("m", 0), case["n"], case["d"], case["k"]
    f32 = case.get("dtype") == "f32"
    code = pm.MEM_F32 if f32 else pm.MEM_BF16
    extra = m if kind == "round" else 0
    s["bank"], s["q"], src = _mixture(g, n, d, m, torch.float32 if f32 else torch.bfloat16, extra)
    if kind == "relations":
        s["out"], s["ws"] = _out(n, k), _bytes(pm.mem_workspace_bytes(n, n, d, k, code))
        return s
    s["out"], s["ws"] = _out(m, k), _bytes(pm.mem_workspace_bytes(m, n + extra, d, k, code))
    if kind == "retrieve":
        s["full"] = torch.empty((m, n), device=DEV) if case["probs"] else None
    if kind == "round":
        s["table"] = torch.arange((n + extra) * case["ppc"], dtype=torch.int32, device=DEV).view(-1, case["ppc"])
    if kind in ("scoped", "request"):
        ns, s["row_ns"] = _namespaces(g, n, case["spaces"], case["burst"])
        s["q_ns"] = ns[src].contiguous()
    if kind in ("step", "request"):
        s["pool"] = _pool(g, case["pages"], case["page"])
        s["table"] = _directory(g, n, case["ppc"], case["pages"])
    if kind == "step":
        s["blocks"] = torch.empty((m * k, case["ppc"], case["page"] // 8), dtype=torch.int64, device=DEV)
    if kind == "request":
        s["offsets"], s["chunks"] = _tables(s["row_ns"], case["spaces"])
        s["ws"] = _bytes(pm.mem_workspace_bytes_grouped(m, case["spaces"], s["chunks"].shape[0], d, k))
        s["tok"] = torch.randint(128, 513, (n,), generator=g, device=DEV, dtype=torch.int32)
        s["prefix"] = (torch.empty((m, case["budget"], 32), dtype=torch.int64, device=DEV),
                       torch.empty((m,), dtype=torch.int32, device=DEV),
                       torch.empty((m, k), dtype=torch.int32, device=DEV))
    return s


def _prepare_maintain(s, g):
    """A pool after a history of updates: block b keeps a uniform share of its pages live, in append order."""
    P, ppc, m, k = s["per_block"], s["ppc"], s["m"], s["k"]
    s["next"] = s["blocks"] * P
    share = torch.rand((s["blocks"], 1), generator=g, device=DEV)
    # (half of all pages, those whose draw lies lowest against their block's share)
    chunks = s["next"] // 2 // ppc
    drawn = torch.rand((s["blocks"], P), generator=g, device=DEV) - share
    live = torch.sort(torch.topk(drawn.flatten(), chunks * ppc, largest=False).indices).values
    s["table0"] = live.view(chunks, ppc).to(torch.int32)
    s["table"] = torch.empty_like(s["table0"])
    ns = torch.randint(0, s["spaces"], (chunks,), generator=g, device=DEV, dtype=torch.int32)
    s["offsets"], s["chunks"] = _tables(ns, s["spaces"])
    # each key's related chunks: a run of neighbours and some further away, scores falling with rank
    near = torch.randint(0, chunks, (m, 1), generator=g, device=DEV)
    step = torch.randint(1, 9, (m, k), generator=g, device=DEV).cumsum(1)
    s["ids"] = ((near + step) % chunks).to(torch.int32)
    s["scores"] = torch.sort(0.5 + 0.5 * torch.rand((m, k), generator=g, device=DEV), dim=1, descending=True).values
    most = s["next"] + m * k * ppc
    s["pool"] = _pool(g, most + P + chunks * ppc + s["spaces"] * P, s["page"])
    most_blocks = (most + P - 1) // P
    s["phi"] = torch.zeros((most_blocks,), device=DEV)
    s["released"] = torch.zeros((most_blocks,), dtype=torch.uint8, device=DEV)
    s["ws_c"] = _bytes(pm.mem_colocate_workspace_bytes(m, k, chunks))
    s["ws_b"] = _bytes(pm.mem_compact_workspace_bytes(most, P, s["chunks"].shape[0], ppc, s["spaces"]))
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "retrieve":
        out = pm.mem_retrieve_topk(s["bank"], s["q"], s["k"], 1.0, out=s["out"], full_prob=s["full"],
                                   workspace=s["ws"])
        return {"topk": out, "full": s["full"]}
    if kind == "relations":
        return {"topk": pm.mem_build_relations(s["bank"], s["k"], 1.0, True, out=s["out"], workspace=s["ws"])}
    if kind == "scoped":
        return {"topk": pm.mem_retrieve_topk_scoped(s["bank"], s["row_ns"], s["q"], s["q_ns"], s["k"], 1.0,
                                                    out=s["out"], workspace=s["ws"])}
    if kind == "step":
        out = pm.mem_retrieve_topk(s["bank"], s["q"], s["k"], 1.0, out=s["out"], workspace=s["ws"])
        blocks = pm.mem_gather_chunks(s["pool"], s["table"], out[0], pm.MEM_ORDER_TIME, s["k"], out=s["blocks"])
        return {"topk": out, "blocks": blocks}
    if kind == "round":
        n, m, ppc = s["n"], s["m"], s["ppc"]
        st = pm.BankState(s["bank"], n, s["table"], n * ppc, (n + m) * ppc)
        out = pm.mem_retrieve_topk(st.live, s["q"], s["k"], 1.0, out=s["out"], workspace=s["ws"])
        pm.mem_append_chunks(st, s["q"])
        return {"topk": out, "rows": st.emb[n:st.n], "table": st.table, "counters": [st.n, st.next_free_page]}
    if kind == "request":
        out = pm.mem_retrieve_topk_grouped(s["bank"], s["offsets"], s["chunks"], s["q"], s["q_ns"], s["k"], 1.0,
                                           out=s["out"], workspace=s["ws"])
        rows, tokens, kept = pm.mem_gather_budget(s["pool"], s["table"], s["tok"], out[0], s["budget"], 256,
                                                  out=s["prefix"])
        return {"topk": out, "rows": rows, "tokens": tokens, "kept": kept}
    s["table"].copy_(s["table0"])
    moved = pm.mem_colocate(s["pool"], s["table"], s["ids"], s["scores"], 0.7, 2, s["next"], workspace=s["ws_c"])
    res, phi, released = pm.mem_compact_blocks(s["pool"], s["table"], s["offsets"], s["chunks"], s["per_block"], 0.3,
                                               moved["next_free_page"], phi=s["phi"], released=s["released"],
                                               workspace=s["ws_b"])
    return {"moved": moved, "compacted": res, "phi": phi, "released": released, "table": s["table"],
            "pool": s["pool"]}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    kind, k = case["kind"], case["k"]
    if kind == "maintain":
        # half the written pages are live, most of them in blocks that are compacted; three fifths of the related
        # chunks are related strongly enough to move
        pages = case["blocks"] * case["per_block"] * 0.4 + case["m"] * k * 0.6 * case["ppc"]
        return {"bytes": 2.0 * pages * case["page"], "flops": 0}
    n, d = case["n"], case["d"]
    size = 4 if case.get("dtype") == "f32" else 2
    m = n if kind == "relations" else case["m"]
    rows = float(n)
    # every pair of a key and a row is one product, except that each key's own namespace holds 1/spaces of the rows,
    # and that a relation build's scores are the same both ways
    pairs = float(m) * n
    if kind == "relations":
        pairs /= 2
    if kind in ("scoped", "request"):
        pairs *= 0.9 / case["spaces"]
        rows *= 0.9 * min(1.0, m / case["spaces"])
    total = size * (rows + (0 if kind == "relations" else m)) * d + 12.0 * m * k + 4.0 * m
    if kind == "retrieve" and case["probs"]:
        total += 4.0 * m * n
    if kind == "step":
        total += 2.0 * m * k * case["ppc"] * case["page"]
    if kind == "round":
        total += 4.0 * m * d
    if kind == "request":
        total += 256.0 * m * (case["budget"] + min(case["budget"], 320 * k))
    return {"bytes": total, "flops": 2.0 * pairs * d}


def tolerance(case):
    """fp32 sums of at most 1,024 products: against 64 bits the results are at most 7e-7 off (norms) and 2.3e-6 (any one
    value), and up to 0.2 % of neighbours in a list are near enough to change places, with the blocks fetched for them."""
    if case["kind"] == "maintain":
        return "exact"
    return {"rel": 3e-6, "max": 1e-5, "differ": 0.01}


# ---------------------------------------------------------------- in 64 bits

def exact(case, seed):
    if case["kind"] == "maintain":
        return None
    s = prepare(case, seed)
    n, k = s["n"], s["k"]
    bank, q = s["bank"][:n], s["bank"][:n] if s["kind"] == "relations" else s["q"]
    probs = s["full"] is not None if s["kind"] == "retrieve" else False
    score, lse, full = [], [], []
    width = min(max(1, (1 << 28) // max(1, q.shape[0] if q.shape[0] < 4096 else 4096)), n)
    for q0 in range(0, q.shape[0], 4096):
        qd = q[q0:q0 + 4096].double()
        best = qd.new_full((qd.shape[0], k), -math.inf)
        total = qd.new_full((qd.shape[0],), -math.inf)
        for r0 in range(0, n, width):
            sc = qd @ bank[r0:r0 + width].double().T
            if s["kind"] == "relations":
                i = torch.arange(q0, q0 + qd.shape[0], device=DEV)
                here = (i >= r0) & (i < r0 + sc.shape[1])
                sc[here.nonzero().flatten(), i[here] - r0] = -math.inf
            if "row_ns" in s:
                rn = s["row_ns"][r0:r0 + width]
                sc.masked_fill_(~((rn[None, :] == s["q_ns"][q0:q0 + 4096, None]) & (rn >= 0)[None, :]), -math.inf)
            total = torch.logaddexp(total, torch.logsumexp(sc, 1))
            best = torch.topk(torch.cat([best, torch.topk(sc, min(k, sc.shape[1]), 1).values], 1), k, 1).values
            if probs:
                full.append(sc)
        score.append(best)
        lse.append(total)
    score, lse = torch.cat(score), torch.cat(lse)
    prob = torch.where(score == -math.inf, 0.0, torch.exp(score - lse[:, None]))
    found = {"topk": [None, score, prob, lse]}
    if probs:
        found["full"] = torch.exp(torch.cat(full, 1) - lse[:, None])
    return found
