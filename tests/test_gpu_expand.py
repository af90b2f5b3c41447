"""Reduction through W on the matrix cores (products of four pairs, a table
of 16 nodes per wavefront, 56 nodes in the workgroup's accumulator) against
the oracle, at list lengths around its units and with rows of W that share
few or no nodes: one to four entries, empty rows, a column twice in a row.
The embedding is kept by the offsets x_off = x - W q.  1e-10, relative, in
global norms: some 500 terms per entry at 1e-16 each, times the cancellation
of the projected blocks (1e3 or less), two decades to spare."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import paper_2409_16385_amd as E  # noqa: E402
from scenes import config1  # noqa: E402

TOL = 1e-10
FLAGS = E.GRAD | E.HESS | E.PROJECT


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


def _rel(a, b):
    n = np.linalg.norm(b)
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / (n if n > 0 else 1.0)


def _rewired(n_node, spread, most=4):
    """config1 with its rows replaced: vertex v has v % (most + 1) entries in
    a window of `spread` nodes; every fifth full row holds a column twice."""
    sc = config1()
    rng = np.random.default_rng(n_node + spread)
    x = O.embed(sc, sc.q)
    n = sc.n_vert
    cnt = np.arange(n) % (most + 1)
    rowptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    col, val = [], []
    for v in range(n):
        w0 = (v * (n_node - spread + 1)) // n
        c = w0 + rng.choice(spread, size=cnt[v], replace=False)
        if cnt[v] == most and most > 1 and v % 5 == 0:
            c[1] = c[0]
        col.extend(c)
        val.extend(rng.uniform(0.1, 1.0, size=cnt[v]))
    col, val = np.array(col, np.int32), np.array(val)
    q = rng.normal(size=3 * n_node) * 1e-2
    y = np.zeros((n, 3))
    np.add.at(y, np.repeat(np.arange(n), cnt), val[:, None] * q.reshape(-1, 3)[col])
    return dataclasses.replace(sc, n_node=n_node, W_rowptr=rowptr, W_col=col, W_val=val, x_off=x - y, q=q,
                               dq=np.zeros(3 * n_node)), x


@pytest.fixture(scope="module")
def ctx():
    return E.Context(0)


@pytest.mark.parametrize("n_node,spread,most", [(1, 1, 1), (16, 16, 4), (17, 17, 4), (57, 57, 4), (400, 300, 4),
                                                (200, 8, 4), (300, 2, 2)])
@pytest.mark.parametrize("hess", ["dense", "bsr"])
def test_reduction_of_rewired_rows(ctx, n_node, spread, most, hess):
    sc, x = _rewired(n_node, spread, most)
    dsc = E.Scene.from_host(ctx, sc)
    pt, ee = O.candidates_grid(sc, O.embed(sc, sc.q), sc.dhat)
    pt = pt[O.narrow(sc, O.embed(sc, sc.q), 0, pt, sc.dhat)[2]]
    ee = ee[O.narrow(sc, O.embed(sc, sc.q), 1, ee, sc.dhat)[2]]
    assert len(pt) > 65 and len(ee) > 60
    for n in (1, 3, 4, 5, 63, 65, max(len(pt), len(ee))):
        p, e = pt[:n], ee[:n]
        r = E.barrier_reduce(ctx, dsc, _dev(sc.q), _dev(p), _dev(e), sc.dhat, sc.kappa, FLAGS, hess=hess)
        ref = O.barrier_reduce(sc, sc.q, p, e, sc.dhat, sc.kappa, FLAGS)
        assert r["n_active"] == ref["n_active"]
        assert _rel(r["grad"].cpu().numpy(), ref["grad"]) <= TOL
        H = r["hess"].cpu().numpy() if hess == "dense" else E.bsr_to_dense(*r["hess"], sc.n_node)
        assert _rel(H, ref["hess"]) <= TOL
    r = E.barrier_reduce(ctx, dsc, _dev(sc.q), _dev(p), _dev(e), sc.dhat, sc.kappa, E.GRAD, hess=None)
    assert _rel(r["grad"].cpu().numpy(), ref["grad"]) <= TOL


def test_a_pair_that_is_not_finite_stays_at_its_nodes():
    """A lagged force that is not finite: the call that reads the status
    reports it; in the other's outputs the nodes of that pair take it, and all
    the other entries are those of the list without the pair."""
    ctx, lam = E.Context(0), np.inf
    sc, x = _rewired(200, 8)
    dsc = E.Scene.from_host(ctx, sc)
    pt, _ = O.candidates_grid(sc, O.embed(sc, sc.q), sc.dhat)
    pt = pt[O.narrow(sc, O.embed(sc, sc.q), 0, pt, sc.dhat)[2]][:30]
    none = np.zeros((0, 2), np.int32)
    st, lag = O.friction_lag_list(sc, sc.q, 0, pt, sc.dhat, sc.kappa, 0)
    assert st == O.OK and (lag[:, 0] > 0).all()
    epsvh = 1e-5
    q = sc.q + np.random.default_rng(0).normal(size=sc.q.shape) * 2e-6
    lag0 = np.zeros((0, lag.shape[1]))
    k = 13
    keep = np.arange(len(pt)) != k
    ref = O.friction_reduce(sc, q, pt[keep], lag[keep], none, lag0, 0.8, epsvh)
    bad = lag.copy()
    bad[k, 0] = lam
    args = (dsc, _dev(q), _dev(pt), _dev(bad), _dev(none), _dev(lag0), 0.8, epsvh)
    r = E.friction_reduce(ctx, *args, hess="dense")
    g = r["grad"].cpu().numpy().reshape(-1, 3)
    H = r["hess"].cpu().numpy()
    with pytest.raises(E.EipcError):
        E.friction_reduce(ctx, *args, hess="bsr")
    H = H.reshape(sc.n_node, 3, sc.n_node, 3).transpose(0, 2, 1, 3)
    v = [pt[k, 0], *sc.faces[pt[k, 1]]]
    nodes = np.unique(np.concatenate([sc.W_col[sc.W_rowptr[i]:sc.W_rowptr[i + 1]] for i in v]))
    own = np.zeros(sc.n_node, bool)
    own[nodes] = True
    assert np.isfinite(g[~own]).all() and _rel(g[~own], ref["grad"].reshape(-1, 3)[~own]) <= TOL
    both = own[:, None] & own[None, :]
    Hr = np.asarray(ref["hess"]).reshape(sc.n_node, 3, sc.n_node, 3).transpose(0, 2, 1, 3)
    assert np.isfinite(H[~both]).all() and _rel(H[~both], Hr[~both]) <= TOL
