"""Launch paths by size, on inputs whose similarities are exact in binary32:
every row has 0 and 255 among integer components (so its step is 1 and its
decoded vector is itself) and queries are small integers, so any order of
summation gives the same value and results equal numpy's, ties to the lower
slot included."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2402_02044_amd as lib
    return lib


def int_rows(g, n, d):
    x = g.integers(0, 256, (n, d)).astype(np.float32)
    x[:, 0], x[:, d - 1] = 0.0, 255.0
    x[n // 2:] = x[g.integers(0, n // 2, n - n // 2)]   # repeats: ties
    return x


def int_queries(g, nq, d):
    return g.integers(-8, 9, (nq, d)).astype(np.float32)


def values(metric_ip, Q, X):
    q, x = Q.astype(np.int64), X.astype(np.int64)
    ip = q @ x.T
    return ip if metric_ip else (q * q).sum(1)[:, None] - 2 * ip + (x * x).sum(1)[None, :]


def best(metric_ip, v, k):
    """(ids, values) of the k best of each row of v, padded."""
    nq, n = v.shape
    key = -v if metric_ip else v
    ids = np.full((nq, k), -1, np.int64)
    val = np.full((nq, k), -np.inf if metric_ip else np.inf)
    for i in range(nq):
        o = np.lexsort((np.arange(n), key[i]))[:k]
        ids[i, :len(o)], val[i, :len(o)] = o, v[i, o]
    return ids, val


def store(L, X, metric_ip, means=None, dead=()):
    ix = L.Index(X.shape[1], 8, 0, L.LVQ_IP if metric_ip else L.LVQ_L2, L.LVQ_SEQUENTIAL, capacity=X.shape[0],
                 means=np.zeros((1, X.shape[1]), np.float32) if means is None else means)
    ix.insert(torch.from_numpy(X).cuda())
    if len(dead):
        ix.delete(torch.tensor(dead, dtype=torch.int32, device="cuda"))
    return ix


@pytest.mark.parametrize("metric_ip,prec", [(True, "bf16"), (True, "fp32"), (False, "fp32")])
@pytest.mark.parametrize("nq,k", [(1, 1), (1, 64), (3, 65), (1, 128), (2, 129), (33, 10), (1, 512), (130, 7)])
def test_topk_merge_edges(L, metric_ip, prec, nq, k):
    """Merges of many parts: one wave per query up to sixteen, lists of one to
    512 keys (each register list length), parts left with fewer than k keys."""
    g = synth.rng(7100 + nq, k)
    n, d = 20_011, 96
    X, Q = int_rows(g, n, d), int_queries(g, nq, d)
    dead = np.unique(g.integers(0, n, 500))
    ix = store(L, X, metric_ip, dead=dead)
    v = values(metric_ip, Q, X)
    v = v.astype(np.float64)
    v[:, dead] = -np.inf if metric_ip else np.inf
    ids, val = best(metric_ip, v, k)
    q = torch.from_numpy(Q).cuda().to(torch.bfloat16 if prec == "bf16" else torch.float32)
    ti, td = ix.topk(q, k)
    assert ix.sync() == 0
    np.testing.assert_array_equal(ti.cpu().numpy(), ids)
    np.testing.assert_array_equal(td.cpu().numpy().astype(np.float64), val)
    ix.close()
