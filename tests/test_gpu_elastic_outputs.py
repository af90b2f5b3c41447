"""Elastic terms with each combination of outputs (the lanes that a tet gets
depend on it): the same sums, and no output that makes another dearer."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_16385_amd as E  # noqa: E402


def _body(m):
    """m^3 nodes of a cube, six tets to a cell, turned and shaken."""
    x = np.arange(m) / (m - 1.0)
    P = np.stack(np.meshgrid(x, x, x, indexing="ij"), -1).reshape(-1, 3)
    c = np.stack(np.meshgrid(*[np.arange(m - 1)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    T = []
    for p in itertools.permutations(range(3)):
        corner = np.zeros((4, 3), int)
        for s in range(3):
            corner[s + 1:, p[s]] += 1
        T.append((c + corner) @ [m * m, m, 1])
    T = np.stack(T, 1).reshape(-1, 4)
    rng = np.random.default_rng(0)
    Q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    Q *= np.sign(np.linalg.det(Q))
    q = P @ Q.T + 0.05 / m * rng.normal(size=P.shape)
    dev = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=t, device="cuda:0")  # noqa: E731
    vol = rng.uniform(0.5, 1.5, len(T)) * (np.arange(len(T)) % 7 > 0)  # some tets are skipped
    return len(P), dev(T, torch.int32), dev(P.reshape(-1)), dev(vol), dev(q.reshape(-1))


def _terms(ctx, body, model, energy, grad, hess):
    n, tets, rest, vol, q = body
    z = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda:0")  # noqa: E731
    out = {"energy": z(1) if energy else None, "grad": z(3 * n) if grad else None,
           "hess": z(3 * n, 3 * n) if hess else None}
    E.elastic(ctx, n, tets, rest, vol, 1e5, 0.3, model, q, 0.7, **out)
    return out


@pytest.mark.parametrize("m", [2, 5, 9])
@pytest.mark.parametrize("model", [E.binding.ELASTIC_LINEAR, E.binding.ELASTIC_COROTATIONAL])
def test_every_combination_of_outputs(m, model):
    """1e-12: sums of the same terms in another order."""
    ctx, body = E.Context(0), _body(m)
    ref = _terms(ctx, body, model, True, True, True)
    assert ctx.sync_status() == E.binding.OK and float(ref["energy"]) > 0
    for want in itertools.product((False, True), repeat=3):
        got = _terms(ctx, body, model, *want)
        for k, t in got.items():
            if t is not None:
                assert float((t - ref[k]).norm()) <= 1e-12 * float(ref[k].norm())


@pytest.mark.parametrize("model", [E.binding.ELASTIC_LINEAR, E.binding.ELASTIC_COROTATIONAL])
def test_an_energy_costs_less_than_a_gradient(model):
    """510,000 tets: a line search asks for the energy alone."""
    ctx, body = E.Context(0), _body(45)

    def ms(*want):
        best = np.inf
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                _terms(ctx, body, model, *want)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        return best

    e, g, eg = ms(True, False, False), ms(False, True, False), ms(True, True, False)
    print(f"energy {e:.4f} ms, gradient {g:.4f}, both {eg:.4f}")
    assert e <= g and eg <= 2 * g
