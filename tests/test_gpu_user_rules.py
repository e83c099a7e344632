"""Which predictor a run-time PDE takes, by its quantities, its source term and
the mesh: Euler with carried densities, with a source term that is zero or
without one, on either side of the rules.

Bar: relative L2 <= 1e-12 against the oracle's step (a few hundred FP64
operations per value, about 1e-14), the carried densities being the same
multiple of the density after the step.
"""
import numpy as np
import pytest

import oracle as O
from paper_1905_07987_amd import adg, inputs
from test_gpu_many_sources import EULER2, dev, rel_l2
from test_gpu_user_pde import EULER3

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ZERO_SOURCE = """template <class R>
  __device__ static void source(const R* Q, R* S) { for (int v = 0; v < NV; ++v) S[v] = R(0) * Q[v]; }
  template <class R>
  __device__ static bool admissible"""


def text(dim, extra, source):
    e = dim + 1
    t = (EULER2 if dim == 2 else EULER3).replace(f"NV = {e + 1}", f"NV = {e + 1 + extra}")
    t = t.replace(f"F[{e}] = ud * (Q[{e}] + p);",
                  f"F[{e}] = ud * (Q[{e}] + p); for (int i = {e + 1}; i < NV; ++i) F[i] = ud * Q[i];")
    t = t.replace(f"lam[{e}] = u + c;", f"lam[{e}] = u + c; for (int i = {e + 1}; i < NV; ++i) lam[i] = u;")
    if source:
        t = t.replace("HAS_SOURCE = false", "HAS_SOURCE = true")
        t = t.replace("template <class R>\n  __device__ static bool admissible", ZERO_SOURCE)
    return t


@pytest.mark.parametrize("dim,order,cells,extra,source", [
    (2, 5, [43, 44], 0, True), (2, 5, [43, 44], 1, True), (2, 5, [43, 44], 1, False),
    (2, 6, [43, 44], 1, True), (2, 6, [43, 44], 2, True), (2, 6, [43, 44], 4, True),
    (2, 7, [43, 44], 0, True), (2, 7, [43, 44], 0, False), (2, 3, [130, 120], 0, True),
    (3, 3, [10, 11, 10], 0, False), (3, 3, [10, 12, 10], 0, True), (3, 3, [5, 4, 4], 1, False),
    (3, 4, [6, 7, 7], 0, True), (3, 4, [9, 9, 9], 0, True), (3, 4, [9, 9, 9], 0, False), (3, 4, [9, 9, 9], 1, True),
    (3, 5, [8, 8, 4], 0, False), (3, 5, [8, 8, 5], 0, False), (3, 5, [8, 8, 5], 0, True)])
def test_against_oracle(dim, order, cells, extra, source):
    print("[gpu-test] user rules", dim, order, cells, dim + 2 + extra, source, flush=True)
    P = O.problem(dim, order, O.EULER, cells, cfl=0.4)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 59)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.0)
    f = 0.5 + 0.7 * np.arange(extra)
    s = adg.Solver(dim, order, "euler", cells, cfl=0.4, source=text(dim, extra, source))
    Q, clock = dev(np.concatenate([Q0, Q0[:, :1] * f[None, :, None]], axis=1)), dev([0.0, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    g = Q.cpu().numpy()
    assert rel_l2(g[:, :dim + 2], Qo) <= 1e-12
    for i in range(extra):
        assert rel_l2(g[:, dim + 2 + i], f[i] * Qo[:, 0]) <= 1e-12
    s.close()


@pytest.mark.parametrize("order,extra", [(5, 2), (5, 3)])
def test_what_did_not_fit_is_refused(order, extra):
    # 7 and 8 quantities at 6^3 nodes exceed the lane pair's shared memory
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, order, "euler", [9, 9, 9], source=text(3, extra, False))
    assert ei.value.status == -5 and "LDS" in str(ei.value)
