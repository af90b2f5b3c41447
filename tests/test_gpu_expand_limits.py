"""The reduction through W where its products could carry a value from one
pair to the nodes of another, and over lists of several steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_16385_amd as E  # noqa: E402
from scenes import scene as S  # noqa: E402


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
