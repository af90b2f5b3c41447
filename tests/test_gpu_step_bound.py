"""The step bound in its two passes (short runs of every pair, then the
undecided ones, few to a wavefront, dropped against the bound published
meanwhile) against the least of the per-pair bounds, which one uninterrupted
run per pair computes: bit for bit, from no undecided pair to many per
wavefront, also where the step cap ends a pair."""
import numpy as np
import pytest
import torch

import paper_2409_16385_amd as E
from paper_2409_16385_amd import batch as BT
from scenes import scene as S

pytestmark = pytest.mark.gpu

SCENES = {
    "tiny": lambda: S.tiny_scene(3),
    "sphere": lambda: S.config1(1),
    "mixed": lambda: S.mixed_scale_scene(0, n=40),
    "grasp": lambda: S.grasp_scene(0, 12, 80, 8, frac=0.7),
}


def _dev(a):
    return None if a is None else torch.as_tensor(np.ascontiguousarray(a), device="cuda:0")


@pytest.mark.parametrize("name", list(SCENES))
@pytest.mark.parametrize("method", [0, 1])
def test_bound_is_the_least_of_the_pairs(name, method):
    sc = SCENES[name]()
    ctx = E.Context(0)
    E.set_ccd_method(ctx, method)
    dsc = E.Scene.from_host(ctx, sc)
    q, dq, off = _dev(sc.q), _dev(sc.dq), _dev(sc.dx_off)
    pt, ee = E.ccd_candidates(ctx, dsc, q, dq, sc.dhat, off)
    steps = 0
    for s in (0.5, 0.1, 1e-3):
        for cap in (1, 4, 5, 9, 100000):
            t = [1.0]
            for kind, p in ((0, pt), (1, ee)):
                if len(p):
                    r = E.ccd_toi(ctx, dsc, q, dq, kind, p, off, s=s, max_iter=cap)
                    t.append(float(r[0].min()))
                    steps = max(steps, int(r[1].max()))
            assert E.ccd_max_step(ctx, dsc, q, dq, sc.dhat, off, s=s, max_iter=cap)[0] == min(t)
    assert steps > 4  # some pair is left to the second pass
