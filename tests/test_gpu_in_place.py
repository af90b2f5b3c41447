"""Outputs that are also inputs: the embedded inputs are read before any
output is cleared, so a product or a gradient may replace its argument."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_16385_amd as E  # noqa: E402
from paper_2409_16385_amd import binding as B  # noqa: E402
from scenes import scene as S  # noqa: E402


def _dev(a):
    return None if a is None else torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


def _same(a, b):
    """Sums of the same terms in another order."""
    return float((a - b).norm()) <= 1e-12 * float(b.norm()) and float(b.norm()) > 0


@pytest.fixture(scope="module")
def case():
    sc = S.tiny_scene(3)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    q = _dev(sc.q)
    return sc, ctx, dsc, q, *E.build_candidates(ctx, dsc, q, sc.dhat)


@pytest.mark.parametrize("noalloc", [False, True])
def test_product_in_place(case, noalloc):
    sc, ctx, dsc, q, pt, ee = case
    rng = np.random.default_rng(0)
    v, v_off = _dev(rng.normal(size=3 * sc.n_node)), _dev(rng.normal(size=(sc.n_vert, 3)))
    ref, ref_off = E.barrier_hvp(ctx, dsc, q, pt, ee, sc.dhat, sc.kappa, E.PROJECT, v, v_off, want_off=True,
                                 noalloc=noalloc)
    L = B._load()
    fn = L.eipc_barrier_hvp_noalloc if noalloc else L.eipc_barrier_hvp
    ctx.check(fn(ctx.handle, dsc.ref, q.data_ptr(), pt.data_ptr(), len(pt), ee.data_ptr(), len(ee), sc.dhat, sc.kappa,
                 E.PROJECT, v.data_ptr(), v_off.data_ptr(), v.data_ptr(), v_off.data_ptr(), ctx.stream()))
    assert _same(v, ref) and _same(v_off, ref_off)


def test_gradient_in_place(case):
    sc, ctx, dsc, q, pt, ee = case
    ref = E.barrier_reduce(ctx, dsc, q, pt, ee, sc.dhat, sc.kappa, E.GRAD, hess=None)["grad"]
    g = q.clone()
    ctx.check(B._load().eipc_barrier_reduce(ctx.handle, dsc.ref, g.data_ptr(), pt.data_ptr(), len(pt), ee.data_ptr(),
                                            len(ee), sc.dhat, sc.kappa, E.GRAD, None, g.data_ptr(), None, None, None,
                                            ctx.stream()))
    assert _same(g, ref)


@pytest.mark.parametrize("with_alpha", [False, True])
def test_planned_gradient_in_place(case, with_alpha):
    sc, _, _, q, _, _ = case
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    dq, off = _dev(sc.dq), _dev(sc.dx_off)
    flags = E.ENERGY | E.GRAD
    plan = E.plan_step(ctx, dsc, q, sc.dhat, dq, off, with_hess=False)
    out = E.StepOut(ctx, dsc, plan, flags, with_alpha=with_alpha)
    E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, dq, off, flags=flags)
    assert ctx.sync_status() == B.OK
    ref = [t.clone() for t in (out.grad, out.energy, out.counts)]
    x = q.clone()
    out.grad = x
    E.contact_step(ctx, dsc, plan, x, sc.dhat, sc.kappa, out, dq, off, flags=flags)
    assert ctx.sync_status() == B.OK
    assert _same(x, ref[0]) and _same(out.energy, ref[1]) and torch.equal(out.counts, ref[2])
