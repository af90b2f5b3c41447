"""The reduction through W where its products could carry a value from one
pair to the nodes of another, and over lists of several steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_16385_amd as E  # noqa: E402
from scenes import config2, scene as S  # noqa: E402


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


def _same(a, b):
    """Sums of the same terms in another order."""
    return float((a - b).norm()) <= 1e-12 * float(b.norm())


def test_hessian_alone_reads_no_stale_gradient():
    """A Hessian without the gradient does not depend on what an earlier call
    left in the records' gradient: neither its values nor its time (a pair
    whose record is not finite is taken alone, a hundred times slower)."""
    sc = S.grasp_scene(0, 36, 500, 16, frac=0.75)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    q = _dev(sc.q)
    pt, ee = E.build_candidates(ctx, dsc, q, sc.dhat)

    def reduction():
        best, hess = np.inf, None
        for _ in range(4):
            ctx.profile_read(reset=True)
            hess = E.barrier_reduce(ctx, dsc, q, pt, ee, sc.dhat, sc.kappa, E.HESS | E.PROJECT)["hess"]
            t = ctx.profile_read(reset=True)
            best = min(best, t["expand_pt"][0] + t["expand_ee"][0])
        return best, hess

    ctx.profile(True)
    t0, h0 = reduction()
    ap, _, ae, _ = E.narrow_phase(ctx, dsc, q, pt, ee, sc.dhat)
    apt, aee = pt[ap.long()].contiguous(), ee[ae.long()].contiguous()
    lpt, lee = E.friction_lag(ctx, dsc, q, apt, aee, sc.dhat, sc.kappa)
    lpt[:, 0] = lee[:, 0] = float("inf")
    E.friction_reduce(ctx, dsc, q + 1e-6, apt, lpt, aee, lee, 0.5, 1e-5, flags=E.GRAD, hess=None)
    ctx.sync_status()
    t1, h1 = reduction()
    ctx.profile(False)
    assert torch.equal(h0[0], h1[0]) and torch.equal(h0[1], h1[1]) and _same(h1[2], h0[2])
    print(f"expansion {t0:.4f} ms, on records with a gradient that is not finite {t1:.4f} ms")
    assert t1 <= 3 * t0


def _two_pairs(w):
    """Two vertices over one triangle, gaps 1e-10 and 5e-3, row v of W being w
    at node v.  Listed 18 and 14 times, so that a wavefront's run of four
    holds both."""
    x = np.array([[0.2, 0.2, 1e-10], [0, 0, 0], [1, 0, 0], [0, 1, 0], [0.5, 0.3, 5e-3]])
    x = x @ np.array([[2, -1, 2], [2, 2, -1], [-1, 2, 2]]) / 3.0  # no axis along the normal
    faces = np.array([[1, 2, 3]], np.int32)
    edges = np.array([[1, 2], [2, 3], [1, 3]], np.int32)
    ctx = E.Context(0)
    sc = E.Scene(ctx, faces, edges, np.arange(6, dtype=np.int32), np.arange(5, dtype=np.int32), np.full(5, w), 5)
    return ctx, sc, _dev((x / w).reshape(-1)), _dev(np.array([[0, 0]] * 18 + [[4, 0]] * 14, np.int32))


@pytest.mark.parametrize("w,kappa", [(1.0, 1.0), (1e8, 1e287), (1e120, 1e58)])
@pytest.mark.parametrize("hess", ["dense", "bsr"])
def test_an_overflow_stays_with_its_pair(w, kappa, hess):
    """Terms of one pair that pass the range in the sums over its rows of W do
    not reach the blocks of another pair's own node."""
    ctx, sc, q, pt = _two_pairs(w)
    none = torch.zeros((0, 2), dtype=torch.int32, device="cuda:0")

    def reduction(pairs):
        r = E.barrier_reduce(ctx, sc, q, pairs, none, 1e-2, kappa, E.GRAD | E.HESS, hess=hess, count=False)
        H = r["hess"].cpu().numpy() if hess == "dense" else E.bsr_to_dense(*r["hess"], 5)
        return r["grad"].cpu().numpy(), H

    (g, H), (g1, H1) = reduction(pt), reduction(pt[18:])
    assert np.isfinite(H[:12, :12]).all() == (w == 1.0)
    big = np.abs(H1[12:]).max()
    assert 0 < big < 1e307
    for a, b in ((H[12:], H1[12:]), (H[:, 12:], H1[:, 12:])):
        assert np.abs(a - b).max() <= 1e-12 * big
    assert np.abs(g[12:] - g1[12:]).max() <= 1e-12 * np.abs(g1[12:]).max()


def test_list_of_several_steps():
    """A wavefront's table, the workgroup's accumulator and their flushes over
    a range of several steps of 1,024 pairs: with one workgroup per CU config
    2's edge pairs are 1,378 to a workgroup.  Against the default launch, one
    step, which the sampled-oracle tests check."""
    sc = config2()
    ctx, ref = E.Context(0), E.Context(0)
    q = _dev(sc.q)
    pt, ee = E.build_candidates(ref, E.Scene.from_host(ref, sc), q, sc.dhat)
    E.set_tuning(ctx, 2.0, [0, 1, 0, 0])
    dsc = E.Scene.from_host(ctx, sc)
    for n in (len(ee), len(ee) - 7777):
        args = (q, pt, ee[:n], sc.dhat, sc.kappa)
        a = E.barrier_reduce(ctx, dsc, *args)
        b = E.barrier_reduce(ref, E.Scene.from_host(ref, sc), *args)
        assert a["n_active"] == b["n_active"] > 350000
        assert torch.equal(a["hess"][0], b["hess"][0]) and torch.equal(a["hess"][1], b["hess"][1])
        assert _same(a["hess"][2], b["hess"][2]) and _same(a["grad"], b["grad"])
        g = E.barrier_reduce(ctx, dsc, *args, flags=E.GRAD, hess=None)["grad"]
        assert _same(g, b["grad"])


@pytest.mark.parametrize("n_node,spread,most", [(16, 16, 4), (57, 57, 4), (400, 300, 4), (3000, 2500, 4)])
@pytest.mark.parametrize("n", [1024 * 256 + 1, 1024 * 256 + 515, 1024 * 768 + 64 * 256])
def test_repeated_list_of_several_steps(n_node, spread, most, n):
    """The same over lists of few and of many nodes (the accumulator of 56 is
    flushed at the end, between steps, or overflows): config 1's pairs listed
    again and again against the sum of their one reduction."""
    from test_gpu_expand import _rewired
    import oracle as O
    sc, x = _rewired(n_node, spread, most)
    pt, _ = O.candidates_grid(sc, x, sc.dhat)
    pt = pt[O.narrow(sc, x, 0, pt, sc.dhat)[2]]
    m, rest = divmod(n, len(pt))
    ctx = E.Context(0)
    E.set_tuning(ctx, 2.0, [0, 1, 0, 0])
    dsc = E.Scene.from_host(ctx, sc)
    q, none = _dev(sc.q), _dev(np.zeros((0, 2), np.int32))
    one, head = _dev(pt), _dev(pt[:rest])
    args = (none, sc.dhat, sc.kappa, E.GRAD | E.HESS | E.PROJECT)
    a = E.barrier_reduce(ctx, dsc, q, torch.cat([one.repeat(m, 1), head]), *args, hess="dense")
    b = E.barrier_reduce(ctx, dsc, q, one, *args, hess="dense")
    c = E.barrier_reduce(ctx, dsc, q, head, *args, hess="dense")
    assert a["n_active"] == n
    for k in ("grad", "hess"):
        assert _same(a[k], m * b[k] + c[k])
    g = E.barrier_reduce(ctx, dsc, q, torch.cat([one.repeat(m, 1), head]), none, sc.dhat, sc.kappa, E.GRAD, hess=None)
    assert _same(g["grad"], m * b["grad"] + c["grad"])
