"""The fused matrix-core pass at the edges of its shapes.  Smaller calls take
the general path, so every case here has at least 2^25 pairs of a query and a
bank row (a relation build at least 2^24): query counts around the three
workgroup shapes, ragged banks, one to five k-blocks per tile, padded rows, the
largest dimension and row stride, every list length, exact ties, namespaces
with fewer rows than a list, and each merge of its partial lists.  Checked
against the oracle on drawn rows."""
import numpy as np
import pytest
import torch

import paper_2607_05708_amd as pm
from paper_2607_05708_amd import inputs
from parity import check_topk, check_topk_scoped

pytestmark = pytest.mark.gpu

TAG = 97


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def up(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(out):
    torch.cuda.synchronize()
    return dict(zip(("idx", "score", "prob", "lse"), (t.cpu().numpy() for t in out)))


def some(m, seed, most=28):
    ends = [0, 63, 64, 127, 128, 255, 256, m - 1]
    return np.unique(np.clip(np.concatenate([ends, np.random.default_rng(seed).integers(0, m, most)]), 0, m - 1))


def sub(g, rows):
    return {key: v[rows] for key, v in g.items()}


# 64 queries take tiles of 64 x 512, 65 to 128 of 128 x 256, more of 256 x 256
@pytest.mark.parametrize("m,n,d,k", [(64, 524289, 32, 16), (65, 516500, 64, 32), (128, 262145, 96, 8), (129, 260200, 160, 17),
                                     (256, 131073, 32, 32), (257, 130700, 64, 1), (1000, 33793, 96, 32),
                                     (2100, 16001, 64, 31), (20000, 1700, 32, 20), (33000, 1025, 128, 16)])
def test_workgroup_shapes(m, n, d, k):
    print(f"case: bf16 m={m} n={n} d={d} k={k}", flush=True)
    cb = inputs.clustered_bank(70, TAG, n, d, 64, 0.3, "bf16", m_queries=m)
    b, q = up(cb.emb), up(cb.queries)
    g = host(pm.mem_retrieve_topk(b, q, k, 2.0))
    rows = some(m, n)
    check_topk(f"fused-{m}-{n}", cb.queries, cb.emb, rows, sub(g, rows), k, 2.0)
    again = host(pm.mem_retrieve_topk(b, q, k, 2.0))
    assert all(np.array_equal(g[key], again[key]) for key in g)


@pytest.mark.parametrize("d,pad", [(160, 24), (32, 8), (96, 0)])
def test_padded_rows(d, pad):
    m, n = 270, 124400
    print(f"case: bf16 m={m} n={n} d={d} rows {pad} and {2 * pad} elements apart", flush=True)
    cb = inputs.clustered_bank(71, TAG, n, d, 64, 0.3, "bf16", m_queries=m)
    b = torch.full((n, d + pad), 7.0, dtype=torch.bfloat16, device="cuda")[:, :d]
    q = torch.full((m, d + 2 * pad), 7.0, dtype=torch.bfloat16, device="cuda")[:, :d]
    b.copy_(up(cb.emb))
    q.copy_(up(cb.queries))
    g = host(pm.mem_retrieve_topk(b, q, 16, 2.0))
    rows = some(m, d)
    check_topk(f"fused-padded-{d}", cb.queries, cb.emb, rows, sub(g, rows), 16, 2.0)


def test_largest_dimension_and_row_stride():
    # 256 k-blocks per tile, bank rows 65,536 elements apart
    m, n, d = 30600, 1100, 8192
    print(f"case: bf16 m={m} n={n} d={d} row stride 65536", flush=True)
    cb = inputs.clustered_bank(72, TAG, n, d, 8, 0.3, "bf16")
    g = torch.Generator(device="cuda").manual_seed(72)
    q = torch.nn.functional.normalize(torch.randn((m, d), generator=g, device="cuda"), dim=1).bfloat16()
    b = torch.zeros((n, 65536), dtype=torch.bfloat16, device="cuda")[:, :d]
    b.copy_(up(cb.emb))
    out = host(pm.mem_retrieve_topk(b, q, 32, 1.0))
    rows = some(m, 72)
    qs = q[torch.from_numpy(rows).cuda()].view(torch.int16).cpu().numpy().view(np.uint16)
    check_topk("fused-d8192", qs, cb.emb, np.arange(len(rows)), sub(out, rows), 32, 1.0)


@pytest.mark.parametrize("k", [5, 16, 32])
def test_exact_ties(k):
    # exactly representable scores, every row twice: ties resolve to the lower ids across tiles and splits
    print(f"case: integer grid m=300 n=120000 d=64 k={k}", flush=True)
    base = inputs.integer_grid(73, TAG, 60000, 64)
    bank = np.concatenate([base, base])
    q = inputs.integer_grid(74, TAG, 300, 64)
    g = host(pm.mem_retrieve_topk(up(bank), up(q), k, 2.0))
    rows = some(300, k)
    check_topk("fused-ties", q, bank, rows, sub(g, rows), k, 2.0, exact=True)


# 20 namespaces, and so many that their rows are fewer than k; merges by workgroups (1,600 partial lists at most) and by waves
@pytest.mark.parametrize("m,n,d,k,spaces", [(64, 530000, 64, 16, 20), (100, 340001, 32, 32, 40000), (300, 112001, 96, 8, 20),
                                            (300, 112001, 32, 32, 12000), (2100, 17000, 64, 32, 20), (2100, 17000, 64, 9, 4000),
                                            (9000, 4097, 32, 32, 900)])
@pytest.mark.parametrize("run", [1, 40])
def test_scoped(m, n, d, k, spaces, run):
    print(f"case: scoped bf16 m={m} n={n} d={d} k={k} namespaces={spaces} run={run}", flush=True)
    cb = inputs.clustered_bank(75, TAG, n, d, 64, 0.3, "bf16", m_queries=m)
    rns, live, kns = inputs.namespaces(75, TAG, n, spaces, 0.1, run=run, query_src=cb.query_src)
    kns = kns.copy()
    kns[::13] = -1
    kns[5::17] = spaces + 3
    g = host(pm.mem_retrieve_topk_scoped(up(cb.emb), up(inputs.scoped_row_ns(rns, live)), up(cb.queries), up(kns), k, 2.0))
    rows = some(m, n)
    check_topk_scoped(f"fused-scoped-{m}", cb.queries, cb.emb, rows, sub(g, rows), k, 2.0, rns, live, kns)
    none = (kns < 0) | (kns >= spaces)
    assert np.all(g["idx"][none] == -1) and np.all(g["lse"][none] == -np.inf)


@pytest.mark.parametrize("n,d,k", [(4097, 32, 8), (4353, 96, 16), (5793, 160, 1), (6145, 64, 32), (8193, 32, 24)])
@pytest.mark.parametrize("own", [True, False])
def test_relation_builds(n, d, k, own):
    # own: each key is left out of its own candidates
    print(f"case: relations bf16 n={n} d={d} k={k} own={own}", flush=True)
    b = inputs.clustered_bank(76, TAG, n, d, 40, 0.3, "bf16").emb
    g = host(pm.mem_build_relations(up(b), k, 2.0, own))
    rows = some(n, k)
    check_topk(f"fused-rel-{n}", b, b, rows, sub(g, rows), k, 2.0, self_idx=np.arange(n) if own else None)
