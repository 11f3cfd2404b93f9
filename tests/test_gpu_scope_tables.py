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
    rows = np.unique(np.concatenate([[0, 63, 64, m - 1], np.random.default_rng(seed).choice(m, 16, replace=False)]))
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
