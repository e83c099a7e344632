"""The FP64 elastic operator with gathered derivatives (orders 1 to 3; at
order 3 the last axis is contracted on the matrix cores): one cell, ragged
last blocks, one Picard iteration and the default, point sources, boundaries;
and a NaN node, which stays in its own cell's results.

Bar: relative L2 <= 1e-12 per field group against the oracle's step (the sums
of the element operator are reordered, each value is a few hundred FP64
operations: about 1e-14).
"""
import numpy as np
import pytest

import oracle as O
from paper_1905_07987_amd import adg, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def setup(order, cells, **kw):
    hi = [500.0 * c for c in cells]
    src = kw.pop("src", None)
    P = O.problem(3, order, O.ELASTIC, cells, [0.0] * 3, hi, sources=[src] if src else (), **kw)
    s = adg.Solver(3, order, "elastic", cells, [0.0] * 3, hi, bc=kw.get("bc"),
                   picard_iters=kw.get("picard_iters") or 0)
    if src:
        s.set_point_sources([src])
    rng = np.random.default_rng(order + 10 * cells[0])
    params = np.column_stack([rng.uniform(2000, 3000, P.ncells), rng.uniform(5000, 7000, P.ncells),
                              rng.uniform(2500, 3400, P.ncells)])
    Q = rng.normal(size=(P.ncells, 9, P.S)) * np.array([6000.0] * 6 + [1.0] * 3)[None, :, None]
    return P, s, Q, params


@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("cells", [[1, 1, 1], [3, 5, 2], [11, 2, 3]])
@pytest.mark.parametrize("iters,source,bc", [(None, False, None), (1, True, None), (None, True, [1, 1, 2, 2, 1, 2])])
def test_steps_against_oracle(order, cells, iters, source, bc):
    print("[gpu-test] linear gather", order, cells, iters, source, bc, flush=True)
    wt = [0.0] * 6 + [0.3, -0.2, 1.0]
    src = dict(x=(230.0, 110.0, 340.0), w=wt, weight=wt, f0=5.0, t0=0.1, amp=1e7) if source else None
    P, s, Q, params = setup(order, cells, src=src, bc=bc, picard_iters=iters)
    dt = 0.5 * O.stable_dt(P, Q, params)[0]
    Qg, prm, clock = dev(Q), dev(params), dev([0.0, dt])
    for k in range(2):
        Q = O.step(P, Q, params, dt, k * dt)
        s.step(Qg, prm, clock, next_dt=False)
    torch.cuda.synchronize()
    g = Qg.cpu().numpy()
    for sl in (slice(0, 6), slice(6, 9)):
        assert np.linalg.norm(g[:, sl] - Q[:, sl]) <= TOL * np.linalg.norm(Q[:, sl])
    s.close()


@pytest.mark.parametrize("order", [1, 2, 3])
def test_nan_stays_in_its_cell(order):
    P, s, Q, params = setup(order, [5, 3, 3])
    Q[7, 2, 1] = np.nan
    Qg = dev(Q)
    out = torch.empty_like(Qg)
    s.predict(Qg, dev(params), dev([0.0, 1e-3]), out)
    torch.cuda.synchronize()
    bad = ~np.isfinite(out.cpu().numpy()).all(axis=(1, 2))
    assert bad[7] and bad.sum() == 1
    s.close()
