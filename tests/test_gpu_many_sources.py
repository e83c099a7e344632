"""As many point sources as the API takes (16), several of them in one cell
and in the last one: every predictor tabulates the sources' amplitudes at its
time nodes in shared memory, and a block can have fewer threads than the table
has entries.

Bar: relative L2 <= 1e-12 against the oracle's step (as for one source: a few
hundred FP64 operations per value, about 1e-14), 1e-5 for the FP32 predictor;
the sources move their cells by far more than that.
"""
import numpy as np
import pytest

import oracle as O
from paper_1905_07987_amd import adg, inputs
from test_gpu_user_pde import EULER3

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EULER2 = (EULER3.replace("DIM = 3, NV = 5", "DIM = 2, NV = 4").replace("Q[4]", "Q[3]").replace("F[4]", "F[3]")
          .replace(" + Q[3] * Q[3])", ")").replace("a < 3", "a < 2").replace("lam[3] = u;", "u;")
          .replace("lam[4]", "lam[3]"))

# NV quantities, each advected on its own, by the non-conservative product
ADVECTION_NCP = r"""
struct AdgUserPDE {
  static constexpr int DIM = 2, NV = 13, NP = 0;
  static constexpr bool LINEAR = false, HAS_NCP = true, HAS_SOURCE = false;
  template <class R>
  __device__ static void flux(const R*, int, R* F) { for (int v = 0; v < NV; ++v) F[v] = R(0); }
  template <class R>
  __device__ static void eigenvalues(const R*, int d, R* lam) {
    for (int v = 0; v < NV; ++v) lam[v] = d == 0 ? R(0.7) : R(-0.4);
  }
  template <class R>
  __device__ static void ncp(const R*, const R* g, R* B) {
    for (int v = 0; v < NV; ++v) B[v] = R(0.7) * g[v] - R(0.4) * g[NV + v];
  }
  template <class R>
  __device__ static bool admissible(const R*) { return true; }
};
"""


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def sixteen(dim, nv, cells, seed):
    """Eight sources for the oracle (its limit), 0 .. 3 of them in the last
    cell and 4 .. 7 in the first two, and the same as sixteen: source s is
    entries s and 15 - s, each with a part of the weights."""
    rng = np.random.default_rng(seed)
    eight, parts = [], [None] * 16
    for s in range(8):
        cell = [c - 1 for c in cells] if s < 4 else [s % 2] + [0] * (dim - 1)
        x = [(c + rng.uniform(0.1, 0.9)) / n for c, n in zip(cell, cells)]
        w = np.array([0.0] + list(rng.uniform(0.1, 0.3, nv - 2) * rng.choice([-1, 1], nv - 2)) + [0.5])
        common = dict(x=x, f0=rng.uniform(1.5, 2.5), t0=rng.uniform(0.05, 0.15),
                      amp=rng.uniform(0.5, 1.0) * 0.4 / np.prod(cells))
        part = rng.uniform(0.3, 0.7)
        eight.append(dict(common, w=list(w)))
        parts[s], parts[15 - s] = dict(common, weight=list(part * w)), dict(common, weight=list((1 - part) * w))
    return eight, parts


def check(dim, order, cells, guess="constant", precision="fp64", source=None):
    print("[gpu-test] 16 sources", dim, order, cells, guess, precision, source is not None, flush=True)
    src, parts = sixteen(dim, dim + 2, cells, 41 + order)
    kw = dict(cfl=0.4, guess=O.GUESS_CERK if guess == "cerk" else 0)
    P = O.problem(dim, order, O.EULER, cells, sources=src, **kw)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 43)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.05)
    Qn = O.step(O.problem(dim, order, O.EULER, cells, **kw), Q0, None, dt, 0.05)
    s = adg.Solver(dim, order, "euler", cells, cfl=0.4, initial_guess=guess, precision=precision, source=source)
    s.set_point_sources(parts)
    Q, clock = dev(Q0), dev([0.05, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    s.close()
    tol = 1e-12 if precision == "fp64" else 1e-5
    last = P.ncells - 1
    for c in (0, last):
        assert rel_l2(Qo[c], Qn[c]) > (1e-5 if precision == "fp64" else 2e-4)
    g = Q.cpu().numpy()
    assert rel_l2(g, Qo) <= tol
    assert rel_l2(g[last], Qo[last]) <= tol and rel_l2(g[:3], Qo[:3]) <= tol


# 2-D: blocks of one wave (N = 7: a mesh of the one-thread-per-node kernel)
CELLS2 = {7: [28, 28]}


@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("guess", ["constant", "cerk"])
def test_two_dimensions(order, guess):
    check(2, order, CELLS2.get(order, [5, 4]), guess)


@pytest.mark.parametrize("order,cells", [(4, [71, 73]), (5, [55, 56]), (6, [71, 73]), (7, [5, 4])])
def test_two_dimensions_other_kernels(order, cells):
    # packed blocks; lane pairs
    check(2, order, cells)


@pytest.mark.parametrize("order,cells", [(1, [4, 3, 2]), (2, [4, 3, 2]), (3, [4, 3, 2]), (3, [9, 9, 9]), (4, [3, 2, 2]),
                                         (4, [7, 8, 7]), (4, [9, 9, 8]), (5, [3, 2, 2])])
def test_three_dimensions(order, cells):
    check(3, order, cells)


@pytest.mark.parametrize("dim,order,cells", [(2, 2, [5, 4]), (2, 4, [5, 4]), (2, 6, [5, 4]), (2, 7, [28, 28]), (2, 7, [5, 4]),
                                             (3, 2, [4, 3, 2]), (3, 3, [4, 3, 2]), (3, 4, [9, 9, 8])])
def test_run_time_pde(dim, order, cells):
    check(dim, order, cells, source=EULER2 if dim == 2 else EULER3)


@pytest.mark.parametrize("dim,order,cells", [(2, 1, [5, 4]), (2, 7, [5, 4]), (3, 3, [4, 3, 2]), (3, 5, [3, 2, 2])])
def test_single_precision(dim, order, cells):
    check(dim, order, cells, precision="fp32")


@pytest.mark.parametrize("order", [5, 6])
def test_lane_pairs_of_many_quantities(order):
    """13 quantities with a non-conservative product: a block of the lane-pair
    kernel holds one cell, fewer threads than the table has entries.  Against
    the oracle's advection, quantity by quantity."""
    cells, nv = [4, 3], 13
    src, parts = sixteen(2, nv, cells, 47 + order)
    P = O.problem(2, order, O.ADVECTION, cells, adv=(0.7, -0.4, 0.0))
    Q0 = np.random.default_rng(48).normal(size=(P.ncells, nv, P.S))
    dt = O.stable_dt(P, Q0[:, :1])[0]
    Qo = np.concatenate([O.step(O.problem(2, order, O.ADVECTION, cells, adv=(0.7, -0.4, 0.0),
                                          sources=[dict(s, w=[s["w"][v]]) for s in src]),
                                np.ascontiguousarray(Q0[:, v:v + 1]), None, dt, 0.05) for v in range(nv)], axis=1)
    s = adg.Solver(2, order, "advection", cells, source=ADVECTION_NCP)
    s.set_point_sources(parts)
    Q, clock = dev(Q0), dev([0.05, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    s.close()
    assert rel_l2(Q.cpu().numpy(), Qo) <= 1e-12
