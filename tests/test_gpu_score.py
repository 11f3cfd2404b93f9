"""The general selection path (scores of a block, then its selection) at the
edges where it can go wrong: tiles of 32, 64 and 128 queries and of 32 and 128
rows, steps of 4,096 scores, one split and several, blocks that a list
resumes from, row tails of every length, rows without 16-byte alignment, and
more equal scores than a step's candidates.  Checked against the oracle under
the parity rules (eps = 2 d 2^-24 |q| |b|), or exactly where scores are exact."""
import numpy as np
import pytest
import torch

import paper_2607_05708_amd as pm
from paper_2607_05708_amd import inputs
from parity import check_topk, check_topk_scoped

pytestmark = pytest.mark.gpu


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


def pick(m, seed=0, most=48):
    if m <= most:
        return np.arange(m)
    return np.unique(np.concatenate([[0, 31, 32, m - 1], np.random.default_rng(seed).choice(m, most, replace=False)]))


# (dtype, m, n, d, k, full probabilities)
SHAPES = [
    ("f32", 1, 1, 1, 1, True),
    ("f32", 1, 31, 3, 7, True),          # a row shorter than 16 bytes
    ("bf16", 5, 33, 7, 33, True),
    ("f32", 33, 4096, 33, 64, True),     # one step, all of it
    ("f32", 32, 4097, 31, 8, True),      # a second step of one row
    ("bf16", 65, 16384, 17, 40, True),   # the largest one-split bank
    ("bf16", 3, 16385, 100, 64, True),   # several splits, then the merge
    ("f32", 40, 33000, 63, 9, False),    # 64-query tiles, odd d
    ("f32", 31, 33001, 130, 64, False),  # 32-query tiles
    ("f32", 129, 16500, 32, 16, False),  # 128-query tiles, the second with one query
    ("bf16", 300, 33000, 64, 64, False),  # whole stages only
    ("bf16", 300, 13000, 135, 33, False),
    ("f32", 1, 70001, 20, 64, False),
    ("f32", 4097, 8200, 8, 64, False),   # two blocks of queries, three of rows: lists resumed
]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_shapes(i):
    dtype, m, n, d, k, full = SHAPES[i]
    print(f"case: {dtype} m={m} n={n} d={d} k={k} full={full}", flush=True)
    b = inputs.iid_unit(70 + i, 98, 0, n, d, dtype)
    q = inputs.iid_unit(70 + i, 98, 4, m, d, dtype)
    fp = torch.empty((m, n), device="cuda") if full else None
    g = host(pm.mem_retrieve_topk(up(b), up(q), k, 3.0, full_prob=fp))
    rows = pick(m, i)
    sub = {key: v[rows] for key, v in g.items()}
    check_topk(f"score-{i}", q, b, rows, sub, k, 3.0)
    if full:
        p = fp.cpu().numpy()
        assert np.allclose(p.sum(axis=1), 1.0, rtol=0, atol=1e-5)
        assert np.array_equal(np.take_along_axis(p, g["idx"].astype(np.int64), 1), g["prob"])


@pytest.mark.parametrize("dtype,m,n,d", [("f32", 70, 33000, 45), ("bf16", 70, 33000, 45), ("bf16", 9, 900, 64)])
def test_rows_without_alignment(dtype, m, n, d):
    # rows begin at any element: odd strides and a base one element in
    b, q = inputs.iid_unit(91, 98, 0, n, d, dtype), inputs.iid_unit(91, 98, 4, m, d, dtype)

    def shifted(a, stride):
        t = up(a)
        flat = torch.zeros(a.shape[0] * stride + 1, dtype=t.dtype, device="cuda")
        view = flat[1:].view(a.shape[0], stride)[:, :d]
        view.copy_(t)
        return view

    g = host(pm.mem_retrieve_topk(shifted(b, d + 2), shifted(q, d + 4), 20, 1.0))
    rows = pick(m)
    check_topk("shifted", q, b, rows, {key: v[rows] for key, v in g.items()}, 20, 1.0)


def test_relation_build_across_blocks():
    # 4,200 keys: two blocks of queries and two of rows, each key left out of its own candidates
    n = 4200
    b = inputs.iid_unit(92, 98, 0, n, 20, "f32")
    g = host(pm.mem_build_relations(up(b), 48, 2.0, True))
    rows = np.unique(np.concatenate([[0, 4095, 4096, n - 1], pick(n)]))
    check_topk("relation-blocks", b, b, rows, {key: v[rows] for key, v in g.items()}, 48, 2.0, self_idx=np.arange(n))


def test_scoped_across_blocks_and_steps():
    n, m, k = 8300, 4100, 40
    b = inputs.iid_unit(93, 98, 0, n, 12, "f32")
    q = inputs.iid_unit(93, 98, 4, m, 12, "f32")
    rns, live, kns = inputs.namespaces(93, 98, n, 40, 0.2, run=16, m=m)
    kns[:3] = -1
    g = host(pm.mem_retrieve_topk_scoped(up(b), up(inputs.scoped_row_ns(rns, live)), up(q), up(kns), k, 2.0))
    rows = pick(m)
    check_topk_scoped("scoped-blocks", q, b, rows, {key: v[rows] for key, v in g.items()}, k, 2.0, rns, live, kns)


@pytest.mark.parametrize("n", [1500, 4096, 9000, 40000])
@pytest.mark.parametrize("k", [1, 8, 64])
def test_ties_and_orders(n, k):
    # exact scores: all equal (the lowest ids win), rising and falling with the row
    b = np.ones((n, 4), np.float32)
    b[:, 1] = np.arange(n)
    b[:, 2] = -np.arange(n)
    q = np.eye(4, dtype=np.float32)
    g = host(pm.mem_retrieve_topk(up(b), up(q), k, 1e-6))
    low, high = np.arange(k), n - 1 - np.arange(k)
    for i, want in enumerate((low, high, low, low)):
        assert np.array_equal(g["idx"][i], want), i
    assert np.array_equal(g["score"][1], high.astype(np.float32))
    assert np.allclose(g["prob"][0], 1.0 / n, rtol=1e-5) and np.allclose(g["lse"][0], np.log(n) + 1e-6, rtol=1e-5)


@pytest.mark.parametrize("m,n,d,k", [(200000, 300, 8, 64), (252000, 4100, 8, 64), (4097, 4097, 20, 33)])
def test_allocation_free_call_of_many_queries(m, n, d, k):
    # (the lists of all 252,000 queries would fill the 128 MiB scratch array: it holds those of 4,096 at a time)
    b, q = up(inputs.iid_unit(94, 98, 0, n, d, "f32")), up(inputs.iid_unit(94, 98, 4, m, d, "f32"))
    want = pm.mem_retrieve_topk(b, q, k, 1.0)
    out = tuple(torch.empty_like(t) for t in want)
    pm.mem_retrieve_topk_noalloc(b, q, k, 1.0, out=out)
    torch.cuda.synchronize()
    for x, y in zip(want, out):
        assert torch.equal(x, y)
    rows = np.unique(np.concatenate([[0, 4095, 4096, m - 1], pick(m)]))
    g = {key: v.cpu().numpy()[rows] for key, v in zip(("idx", "score", "prob", "lse"), out)}
    check_topk(f"noalloc-{m}", q.cpu().numpy(), b.cpu().numpy(), rows, g, k, 1.0)


# (m, n, k): the calls next to the lines between the fused and the general path
@pytest.mark.parametrize("m,n,k", [(96, 65535, 8), (96, 65536, 8), (63, 262144, 20), (65, 262144, 20),
                                   (1000, 33000, 32), (1100, 33000, 32)])
def test_both_sides_of_the_path_rule(m, n, k):
    cb = inputs.clustered_bank(95, 98, n, 32, 64, 0.3, "bf16", m_queries=m)
    g = host(pm.mem_retrieve_topk(up(cb.emb), up(cb.queries), k, 1.0))
    rows = pick(m, most=24)
    check_topk(f"rule-{m}-{n}", cb.queries, cb.emb, rows, {key: v[rows] for key, v in g.items()}, k, 1.0)


@pytest.mark.parametrize("n,k", [(4096, 5), (4097, 5), (5400, 20), (5700, 5), (5700, 32), (5900, 5), (5900, 32)])
def test_both_sides_of_the_path_rule_for_relations(n, k):
    b = inputs.clustered_bank(96, 98, n, 64, 32, 0.3, "bf16").emb
    g = host(pm.mem_build_relations(up(b), k, 1.0, True))
    rows = pick(n, most=24)
    check_topk(f"rule-rel-{n}", b, b, rows, {key: v[rows] for key, v in g.items()}, k, 1.0, self_idx=np.arange(n))


@pytest.mark.parametrize("d,k", [(776, 40), (800, 8)])
def test_long_rows_of_a_large_bank(d, k):
    # over 1 GiB of rows of 1.5 KiB or more: loaded non-temporally, the last stage not a whole one
    n, m = 700001, 3
    g = torch.Generator(device="cuda").manual_seed(97)
    b = torch.nn.functional.normalize(torch.randn((n, d), generator=g, device="cuda"), dim=1).bfloat16()
    q = torch.nn.functional.normalize(torch.randn((m, d), generator=g, device="cuda"), dim=1).bfloat16()
    idx, score, prob, lse = pm.mem_retrieve_topk(b, q, k, 1.0)
    s = torch.cat([q.double() @ part.double().T for part in b.split(100000)], 1)
    eps = 2.0 * d * 2.0 ** -24 * 1.02  # norms after rounding to bf16
    best = torch.topk(s, k, 1).values
    assert (score.double() - best).abs().max() <= eps
    assert (torch.gather(s, 1, idx.long()) - score.double()).abs().max() <= eps
    assert all(len(set(row)) == k for row in idx.tolist())
    assert (lse.double() - torch.logsumexp(s, 1)).abs().max() <= eps + 1e-5 * 14


# (dtype, m, n, d): tiles of 32 and 64 queries for more queries than one of them holds, next to the tile counts (256) at
# which they begin, the last tile with one query or row
@pytest.mark.parametrize("dtype,m,n,d", [("bf16", 33, 16257, 40), ("bf16", 64, 16385, 200), ("f32", 65, 10881, 20),
                                         ("f32", 97, 8100, 70), ("bf16", 129, 10880, 24), ("bf16", 129, 10881, 72),
                                         ("bf16", 200, 4607, 64), ("f32", 257, 6530, 36), ("bf16", 1025, 1921, 96)])
def test_tiles_of_fewer_queries(dtype, m, n, d):
    print(f"case: {dtype} m={m} n={n} d={d}", flush=True)
    b, q = inputs.iid_unit(99, 98, 0, n, d, dtype), inputs.iid_unit(99, 98, 4, m, d, dtype)
    g = host(pm.mem_retrieve_topk(up(b), up(q), 12, 2.0))
    rows = np.unique(np.concatenate([[0, 31, 32, m - 2, m - 1], pick(m, n)]))
    check_topk(f"tiles-{m}-{n}", q, b, rows, {key: v[rows] for key, v in g.items()}, 12, 2.0)


# (m, n, k): 17, 31 and 32 lists of 32 and 33 and 64 of 16 per query, which one wave merges (up to 64 lists of 1,024 keys
# in all), then 33 of 32 and 68 of 8
@pytest.mark.parametrize("m,n,k", [(60, 69632, 17), (33, 126976, 31), (32, 131072, 32), (31, 135000, 9), (16, 262144, 16),
                                   (31, 135168, 32), (15, 278528, 8)])
@pytest.mark.parametrize("scoped", [False, True])
def test_merges_around_1024_keys(m, n, k, scoped):
    print(f"case: f32 m={m} n={n} k={k} scoped={scoped}", flush=True)
    b, q = inputs.iid_unit(100, 98, 0, n, 8, "f32"), inputs.iid_unit(100, 98, 4, m, 8, "f32")
    rows = np.arange(0, m, 3)
    if not scoped:
        g = host(pm.mem_retrieve_topk(up(b), up(q), k, 2.0))
        check_topk(f"merge-{m}", q, b, rows, {key: v[rows] for key, v in g.items()}, k, 2.0)
        return
    # most namespaces hold fewer rows than there are lists, some fewer than k
    rns, live, kns = inputs.namespaces(100, 98, n, 9000, 0.1, run=3, m=m)
    g = host(pm.mem_retrieve_topk_scoped(up(b), up(inputs.scoped_row_ns(rns, live)), up(q), up(kns), k, 2.0))
    check_topk_scoped(f"merge-scoped-{m}", q, b, rows, {key: v[rows] for key, v in g.items()}, k, 2.0, rns, live, kns)


@pytest.mark.parametrize("d", [1, 4])
def test_full_probabilities_of_half_a_billion_rows(d):
    # 2^24 and more blocks of 32 rows, past the threads of one launch
    n = (1 << 29) + 37
    g = torch.Generator(device="cuda").manual_seed(101)
    b = torch.randn((n, d), generator=g, device="cuda")
    q = torch.zeros((1, d), device="cuda")
    q[0, d - 1] = 1.0
    s = b[:, d - 1]
    full = torch.empty((1, n), device="cuda")
    idx, score, prob, lse = pm.mem_retrieve_topk(b, q, 3, 1.0, full_prob=full)
    top = max((v, -int(i) - r0) for r0 in range(0, n, 1 << 27)
              for v, i in [tuple(x.item() for x in s[r0:r0 + (1 << 27)].max(0))])
    assert idx[0, 0].item() == -top[1] and score[0, 0].item() == top[0]
    assert torch.equal(s[idx[0].long()], score[0])
    total = sum(part.double().exp().sum() for part in s.split(1 << 27)).log()
    assert abs(lse.item() - total.item()) <= 2e-6 * total.item()
    for r0 in (0, (1 << 28) - 50, (1 << 29) - 50, n - 100):
        part = slice(r0, r0 + 100)
        assert torch.allclose(full[0, part].double(), (s[part].double() - total).exp(), rtol=1e-4, atol=0)
    assert abs(sum(part.double().sum() for part in full[0].split(1 << 27)).item() - 1.0) <= 1e-4
