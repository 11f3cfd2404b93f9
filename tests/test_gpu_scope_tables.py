"""Scoped retrievals large enough to collect their namespaces' rows into
chunk tables on the device: namespace ids of any size, namespaces without
rows or without queries, queries without a namespace, ragged sizes, every
list length, few namespaces (where the device keeps the masked pass), and the
same call captured and replayed with other namespaces in place."""
import numpy as np
import pytest
import torch

import paper_2607_05708_amd as pm
from paper_2607_05708_amd import inputs
from parity import check_topk_scoped

pytestmark = pytest.mark.gpu


def up(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bank_of(seed, rows, d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.nn.functional.normalize(torch.randn((rows, d), generator=g, device="cuda"), dim=1).bfloat16()
    return x, x.view(torch.int16).cpu().numpy().view(np.uint16)


def check(name, b, q, rns, live, kns, out, k, seed):
    torch.cuda.synchronize()
    g = dict(zip(("idx", "score", "prob", "lse"), (t.cpu().numpy() for t in out)))
    m = q.shape[0]
    some = np.random.default_rng(seed).choice(m, min(m, 16), replace=False)
    rows = np.unique(np.concatenate([[0, min(63, m - 1), min(64, m - 1), m - 1], some]))
    check_topk_scoped(name, q, b, rows, {key: v[rows] for key, v in g.items()}, k, 1.0, rns, live, kns)
    return g


# (queries, rows, d, k, namespaces, mean run): the masked pass's share of work decides; 3 namespaces keep it
CASES = [
    (4096, 65600, 1024, 32, 200, 1),
    (4095, 65537, 1024, 5, 3000, 16),    # lists of 8: no sample in either pass
    (1023, 300001, 1024, 16, 70, 64),    # lists of 16; about two splits per table
    (2048, 140000, 1024, 17, 1, 8),      # one namespace: declined
    (2048, 140000, 1024, 8, 3, 8),       # declined
    (4096, 8200, 8192, 32, 64, 8),       # the shortest tables and the largest dimension
    # tables that are too many scores (12 * 2^20) or too long (32,768 rows) to be scored first: the fused grouped pass
    # runs over them, in as many splits as the device plans
    (2048, 140000, 1024, 32, 8, 16),
    (2048, 140000, 1024, 6, 9, 1),
    (1024, 300001, 1024, 16, 8, 64),
    (3000, 90001, 1024, 12, 11, 300),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_tables_against_oracle(i):
    m, n, d, k, n_ns, run = CASES[i]
    print(f"case: scope tables m={m} n={n} d={d} k={k} namespaces={n_ns} run={run}", flush=True)
    bt, b = bank_of(60 + i, n, d)
    qt, q = bank_of(160 + i, m, d)
    rns, live, kns = inputs.namespaces(60 + i, 99, n, n_ns, 0.1, run=run, m=m)
    # ids far apart, many in one hash slot's neighbourhood, one at the top of the range
    spread = np.where(np.arange(n_ns) % 2 == 0, np.arange(n_ns) * 8192, 2147483647 - np.arange(n_ns)).astype(np.int64)
    rns, kns = spread[rns].astype(np.int32), spread[kns].astype(np.int32)
    kns[5::97] = -1          # no namespace
    kns[7::101] = 1234567    # one without rows
    out = pm.mem_retrieve_topk_scoped(bt, up(inputs.scoped_row_ns(rns, live)), qt, up(kns), k, 1.0)
    g = check(f"tables-{i}", b, q, rns, live, kns, out, k, i)
    none = (kns == -1) | (kns == 1234567)
    assert np.all(g["idx"][none] == -1) and np.all(g["lse"][none] == -np.inf)


def test_captured_call_follows_the_namespaces():
    # one graph, replayed with namespaces that take the tables and then with one that does not
    m, n, d, k = 2048, 140000, 1024, 12
    bt, b = bank_of(71, n, d)
    qt, q = bank_of(171, m, d)
    many = inputs.namespaces(71, 99, n, 150, 0.1, run=16, m=m)
    one = (np.zeros(n, np.int32), many[1], np.zeros(m, np.int32))
    row_ns, key_ns = up(inputs.scoped_row_ns(many[0], many[1])), up(many[2])
    out = (torch.empty((m, k), dtype=torch.int32, device="cuda"), torch.empty((m, k), device="cuda"),
           torch.empty((m, k), device="cuda"), torch.empty(m, device="cuda"))
    ws = torch.empty(pm.mem_workspace_bytes(m, n, d, k, pm.MEM_BF16), dtype=torch.uint8, device="cuda")

    def call():
        pm.mem_retrieve_topk_scoped(bt, row_ns, qt, key_ns, k, 1.0, out=out, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep, (rns, live, kns) in enumerate((many, one, many)):
        row_ns.copy_(up(inputs.scoped_row_ns(rns, live)))
        key_ns.copy_(up(kns))
        ws.fill_(255)
        graph.replay()
        check(f"replay-{rep}", b, q, rns, live, kns, out, k, rep)


def test_captured_call_over_long_tables():
    # the same for tables that the fused grouped pass takes, in turn with the other two ways
    m, n, d, k = 2048, 140000, 1024, 10
    bt, b = bank_of(72, n, d)
    qt, q = bank_of(172, m, d)
    few, many = (inputs.namespaces(72, 99, n, spaces, 0.1, run=16, m=m) for spaces in (8, 150))
    one = (np.zeros(n, np.int32), many[1], np.zeros(m, np.int32))
    row_ns, key_ns = up(inputs.scoped_row_ns(few[0], few[1])), up(few[2])
    out = (torch.empty((m, k), dtype=torch.int32, device="cuda"), torch.empty((m, k), device="cuda"),
           torch.empty((m, k), device="cuda"), torch.empty(m, device="cuda"))
    ws = torch.empty(pm.mem_workspace_bytes(m, n, d, k, pm.MEM_BF16), dtype=torch.uint8, device="cuda")

    def call():
        pm.mem_retrieve_topk_scoped(bt, row_ns, qt, key_ns, k, 1.0, out=out, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep, (rns, live, kns) in enumerate((few, many, few, one, few)):
        row_ns.copy_(up(inputs.scoped_row_ns(rns, live)))
        key_ns.copy_(up(kns))
        ws.fill_(255)
        graph.replay()
        check(f"long-replay-{rep}", b, q, rns, live, kns, out, k, rep)


def grouped_check(lengths, counts, d, k, seed, n_extra=0):
    """Grouped retrieval with tables of these lengths and these many queries each (interleaved rows and queries)."""
    n = sum(lengths) + n_extra
    m = sum(counts)
    rng = np.random.default_rng(seed)
    bt, b = bank_of(seed, n, d)
    qt, q = bank_of(seed + 100, m, d)
    rns = np.concatenate([np.repeat(np.arange(len(lengths)), lengths), np.full(n_extra, -1)]).astype(np.int32)
    rng.shuffle(rns)
    kns = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    rng.shuffle(kns)
    offsets = np.zeros(len(lengths) + 1, np.int32)
    offsets[1:] = np.cumsum(lengths)
    live = np.nonzero(rns >= 0)[0]
    chunks = live[np.argsort(rns[live], kind="stable")].astype(np.int32)
    out = pm.mem_retrieve_topk_grouped(bt, up(offsets), up(chunks), qt, up(kns), k, 1.0)
    check(f"grouped-{seed}", b, q, rns, (rns >= 0).astype(np.uint8), kns, out, k, seed)


@pytest.mark.parametrize("d,k", [(96, 32), (160, 7), (1024, 16)])
def test_grouped_tile_and_step_edges(d, k):
    # tables around the 128-row tile and the 4,096-score step, queries around the tile of 32
    lengths = [0, 1, 2, 127, 128, 129, 4095, 4096, 4097, 5, 8193]
    counts = [3, 1, 33, 32, 31, 65, 2, 1, 40, 0, 3]
    grouped_check(lengths, counts, d, k, 80, n_extra=11)


@pytest.mark.parametrize("length,queries", [(24576, 512), (24577, 512), (32768, 4), (32769, 4)])
def test_both_sides_of_the_table_rule(length, queries):
    # 12 * 2^20 scores and tables of 32,768 rows are the most that are scored first and selected from after
    grouped_check([length, 300], [queries, 0], 96, 10, 90 + queries % 7)


# (queries, namespaces, rows, d, k): on either side of the size (12 * 2^20 scores of average tables, or their 32,768 rows)
# up to which the tables are given room to be scored first; past it the fused pass alone runs, over queries put in grouped order
@pytest.mark.parametrize("m,n_ns,n,d,k", [(1024, 16, 196600, 96, 12), (1024, 16, 196640, 96, 12), (1024, 16, 393400, 96, 12),
                                          (300, 2, 180001, 128, 32), (250, 8, 410000, 96, 5), (70, 2, 65536, 96, 7), (70, 2, 65538, 96, 7),
                                          (9, 1, 54000, 96, 16)])
def test_grouped_few_long_tables(m, n_ns, n, d, k):
    print(f"case: grouped m={m} namespaces={n_ns} n={n} d={d} k={k}", flush=True)
    bt, b = bank_of(120 + n_ns, n, d)
    qt, q = bank_of(220 + n_ns, m, d)
    rng = np.random.default_rng(n)
    rns = rng.integers(0, n_ns, n).astype(np.int32)
    kns = rng.integers(0, n_ns, m).astype(np.int32)
    kns[::31] = -1           # no namespace
    kns[7::53] = n_ns + 5    # one past the tables
    offsets = np.zeros(n_ns + 1, np.int32)
    offsets[1:] = np.cumsum(np.bincount(rns, minlength=n_ns))
    chunks = np.argsort(rns, kind="stable").astype(np.int32)
    out = pm.mem_retrieve_topk_grouped(bt, up(offsets), up(chunks), qt, up(kns), k, 1.0)
    g = check(f"few-{n}", b, q, rns, np.ones(n, np.uint8), kns, out, k, n_ns)
    none = (kns < 0) | (kns >= n_ns)
    assert np.all(g["idx"][none] == -1) and np.all(g["lse"][none] == -np.inf)
    # every other query was scored: k distinct rows, all of its own namespace
    assert np.all(rns[g["idx"][~none]] == kns[~none, None])
    assert all(len(set(r)) == k for r in g["idx"][~none].tolist())


@pytest.mark.parametrize("repeats,k", [(1500, 5), (3000, 32), (6000, 16)])
def test_table_that_repeats_a_row(repeats, k):
    # outside the contract (a table lists distinct rows): more equal keys than a selection step holds stay within its
    # memory, the row still comes first, and the other namespaces' results are right
    print(f"case: grouped table with {repeats} equal entries k={k}", flush=True)
    n, d, m = 9000, 96, 40
    bt, b = bank_of(130, n, d)
    q = b[4000:4001].repeat(m, 0)           # row 4,000 scores highest for every query
    q[1::2] = b[5000 + np.arange(1, m, 2)]  # (odd queries ask in the other namespace)
    kns = (np.arange(m) % 2).astype(np.int32)
    mine = np.sort(np.concatenate([np.full(repeats, 4000), np.arange(100, 400)])).astype(np.int32)
    other = np.arange(4500, 9000).astype(np.int32)
    offsets = np.array([0, len(mine), len(mine) + len(other)], np.int32)
    out = pm.mem_retrieve_topk_grouped(bt, up(offsets), up(np.concatenate([mine, other])), up(q), up(kns), k, 1.0)
    torch.cuda.synchronize()
    g = dict(zip(("idx", "score", "prob", "lse"), (t.cpu().numpy() for t in out)))
    assert np.all(g["idx"][0::2, 0] == 4000)
    assert set(np.unique(g["idx"][0::2])) <= {-1, 4000} | set(range(100, 400))
    assert np.all(np.isfinite(g["lse"]))
    rows = np.arange(1, m, 2)
    rns = np.where(np.arange(n) >= 4500, 1, 0).astype(np.int32)
    check_topk_scoped(f"repeats-{repeats}", q, b, rows, {key: v[rows] for key, v in g.items()}, k, 1.0, rns,
                      np.ones(n, np.uint8), kns)
