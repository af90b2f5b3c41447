"""Lists and tables at the limits of their sizes: what does not fit is
reported or run again, and nothing past it is read."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_16385_amd as E  # noqa: E402
from paper_2409_16385_amd import binding as B  # noqa: E402
from scenes import scene as S  # noqa: E402

FLAGS = E.ENERGY | E.GRAD | E.HESS | E.PROJECT


def _dev(a):
    return None if a is None else torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


def _same(a, b):
    """Sums of the same terms in another order."""
    return float((a - b).norm()) <= 1e-12 * float(b.norm())


def test_more_blocks_than_the_first_size():
    """A per-call reduction sizes its BSR view from the node count (16 blocks
    a row and 1,024) on a context's first call and is compacted again when
    they are more."""
    sc = S.grasp_scene(0, 50, 400, 28, frac=0.8)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    q = _dev(sc.q)
    pt, ee = E.build_candidates(ctx, dsc, q, sc.dhat)
    dense = E.barrier_reduce(ctx, dsc, q, pt, ee, sc.dhat, sc.kappa, FLAGS, hess="dense")["hess"]
    for _ in range(2):
        rp, col, blk = E.barrier_reduce(ctx, dsc, q, pt, ee, sc.dhat, sc.kappa, FLAGS, hess="bsr")["hess"]
        assert blk.shape[0] > 16 * sc.n_node + 1024
        row = torch.repeat_interleave(torch.arange(sc.n_node, device="cuda:0"), (rp[1:] - rp[:-1]).long())
        at = dense.view(sc.n_node, 3, sc.n_node, 3).permute(0, 2, 1, 3)[row, col.long()]
        assert _same(blk, at) and _same(blk.norm(), dense.norm())


@pytest.mark.parametrize("reserve", [0, 1 << 29])
def test_blocks_past_the_plan(reserve):
    """A plan with fewer BSR blocks than the step has: the overflow is
    reported, rows within the capacity are whole, the row that crosses it
    holds zero blocks."""
    sc = S.config1(0)
    ctx = E.Context(0, reserve_bytes=reserve)
    dsc = E.Scene.from_host(ctx, sc)
    q = _dev(sc.q)
    plan = E.plan_step(ctx, dsc, q, sc.dhat)
    out = E.StepOut(ctx, dsc, plan, FLAGS, with_alpha=False)
    E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, flags=FLAGS)
    assert ctx.sync_status() == B.OK
    rp, col, blk = out.hess(ctx)
    n = (rp[1:] - rp[:-1]).cpu().numpy()
    for r in (int(np.flatnonzero(n > 1)[0]), int(np.flatnonzero(n > 1)[-1])):
        b = int(rp[r])
        plan.nnzb = b + 1
        E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, flags=FLAGS)
        assert ctx.sync_status() == B.ERR_CAPACITY
        rp1, col1, blk1 = out.hess(ctx)
        assert torch.equal(rp1, rp.clamp(max=b + 1)) and torch.equal(col1[:b], col[:b])
        assert b == 0 or _same(blk1[:b], blk[:b])
        assert int(col1[b]) == 0 and not bool(blk1[b].any())


@pytest.mark.parametrize("reserve", [0, 1 << 29])
@pytest.mark.parametrize("buckets", [1, 2, 64])
def test_few_hash_buckets(reserve, buckets):
    """Any power of two of buckets gives the same step, on scratch that an
    earlier call left full of set bits (the empty keys of a block table)."""
    sc = S.tiny_scene(3)
    ctx = E.Context(0, reserve_bytes=reserve)
    dsc = E.Scene.from_host(ctx, sc)
    q, dq, off = _dev(sc.q), _dev(sc.dq), _dev(sc.dx_off)
    plan = E.plan_step(ctx, dsc, q, sc.dhat, dq, off)
    out = E.StepOut(ctx, dsc, plan, FLAGS)

    def step():
        E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, dq, off, flags=FLAGS)
        assert ctx.sync_status() == B.OK
        return [t.clone() for t in (out.counts, out.alpha, out.energy, out.grad)], out.hess(ctx)

    ref, href = step()
    assert int(ref[0][2]) > 0
    none = torch.zeros((0, 2), dtype=torch.int32, device="cuda:0")
    E.barrier_reduce(ctx, dsc, q, none, none, sc.dhat, sc.kappa, FLAGS, hess="bsr")
    for k in range(4):
        plan.buckets[k] = buckets
    for _ in range(2):
        got, hgot = step()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
        assert _same(got[2], ref[2]) and _same(got[3], ref[3])
        assert torch.equal(hgot[0], href[0]) and torch.equal(hgot[1], href[1]) and _same(hgot[2], href[2])


@pytest.mark.parametrize("cap", [0, 5])
@pytest.mark.parametrize("field", ["cand_pt", "cand_ee", "swept_pt", "swept_ee"])
def test_candidates_past_the_plan(field, cap):
    """A list with less room than candidates, or with none, is reported, and
    its count is what it holds."""
    sc = S.tiny_scene(3)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    q, dq, off = _dev(sc.q), _dev(sc.dq), _dev(sc.dx_off)
    plan = E.plan_step(ctx, dsc, q, sc.dhat, dq, off)
    swept = field.startswith("swept")
    out = E.StepOut(ctx, dsc, plan, FLAGS, with_alpha=swept)
    at = ["cand_pt", "cand_ee", "", "swept_pt", "swept_ee"].index(field)
    E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, dq, off, flags=FLAGS)
    assert ctx.sync_status() == B.OK and int(out.counts[at]) > 5
    setattr(plan, field, cap)
    E.contact_step(ctx, dsc, plan, q, sc.dhat, sc.kappa, out, dq, off, flags=FLAGS)
    assert ctx.sync_status() == B.ERR_CAPACITY
    assert int(out.counts[at]) == cap


@pytest.mark.parametrize("swept", [False, True])
def test_nothing_written_when_a_list_does_not_fit(swept):
    """Also on a context's first call, whose first pass over so small a cell
    runs out of hash entries and finds only some of the pairs."""
    import ctypes as C
    sc = S.config1(0)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    q, dq, off = _dev(sc.q), _dev(sc.dq), _dev(sc.dx_off)
    if swept:
        pt, ee = E.ccd_candidates(ctx, dsc, q, dq, sc.dhat, off)
    else:
        pt, ee = E.build_candidates(ctx, dsc, q, sc.dhat)
    ctx = E.Context(0)
    dsc = E.Scene.from_host(ctx, sc)
    E.set_tuning(ctx, 0.4)
    bpt = torch.full((len(pt) - 1, 2), -7, dtype=torch.int32, device="cuda:0")
    bee = torch.full((len(ee) - 1, 2), -7, dtype=torch.int32, device="cuda:0")
    n_pt, n_ee = C.c_int64(), C.c_int64()
    L = B._load()
    lists = (bpt.data_ptr(), len(bpt), bee.data_ptr(), len(bee), C.byref(n_pt), C.byref(n_ee), ctx.stream())
    if swept:
        st = L.eipc_ccd_candidates(ctx.handle, dsc.ref, q.data_ptr(), dq.data_ptr(),
                                   None if off is None else off.data_ptr(), sc.dhat, *lists)
    else:
        st = L.eipc_build_candidates(ctx.handle, dsc.ref, q.data_ptr(), sc.dhat, *lists)
    torch.cuda.synchronize()
    assert st == B.ERR_CAPACITY and (n_pt.value, n_ee.value) == (len(pt), len(ee))
    assert bool((bpt == -7).all()) and bool((bee == -7).all())
