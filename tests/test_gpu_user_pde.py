"""PDEs given as HIP source text (adg_create_user), compiled at run time.

The test writes Euler, elasticity and the advection-decay PDE as user
structs (the pointwise terms of the paper's Table 2) and checks the compiled
step against the oracle (relative L2 <= 1e-12, FP64) and against the
built-in PDEs; a mixed-precision run against the built-in's; the
admissibility check; compile errors (status COMPILE with the compiler's
log) and the refusals (wrong DIM, walls, adjoint).
"""
import numpy as np
import pytest

import oracle as O
from paper_1905_07987_amd import adg, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12

EULER3 = r"""
struct AdgUserPDE {
  static constexpr int DIM = 3, NV = 5, NP = 0;
  static constexpr bool LINEAR = false, HAS_NCP = false, HAS_SOURCE = false;
  template <class R>
  __device__ static R pressure(const R* Q) {
    return R(0.4) * (Q[4] - R(0.5) * (Q[1] * Q[1] + Q[2] * Q[2] + Q[3] * Q[3]) / Q[0]);
  }
  template <class R>
  __device__ static void flux(const R* Q, int d, R* F) {
    const R p = pressure(Q), ud = Q[1 + d] / Q[0];
    F[0] = Q[1 + d];
    for (int a = 0; a < 3; ++a) F[1 + a] = ud * Q[1 + a];
    F[1 + d] += p;
    F[4] = ud * (Q[4] + p);
  }
  template <class R>
  __device__ static void eigenvalues(const R* Q, int d, R* lam) {
    const R u = Q[1 + d] / Q[0], c = sqrt(R(1.4) * pressure(Q) / Q[0]);
    lam[0] = u - c;
    lam[1] = lam[2] = lam[3] = u;
    lam[4] = u + c;
  }
  template <class R>
  __device__ static bool admissible(const R* Q) { return Q[0] > R(0) && pressure(Q) > R(0); }
};
"""

# velocity-stress elasticity: Q = (sxx, syy, szz, sxy, sxz, syz, rho vx, rho vy, rho vz | rho, cp, cs)
ELASTIC = r"""
struct AdgUserPDE {
  static constexpr int DIM = 3, NV = 9, NP = 3;
  static constexpr bool LINEAR = true, HAS_NCP = true, HAS_SOURCE = false;
  __device__ static int sym(int i, int d) { return i == d ? i : (i + d == 1 ? 3 : (i + d == 2 ? 4 : 5)); }
  template <class R>
  __device__ static void flux(const R* Q, int d, R* F) {
    for (int v = 0; v < 6; ++v) F[v] = R(0);
    for (int i = 0; i < 3; ++i) F[6 + i] = Q[sym(i, d)];
  }
  template <class R>
  __device__ static void eigenvalues(const R* Q, int d, R* lam) {
    const R cp = Q[10], cs = Q[11];
    lam[0] = -cp; lam[1] = cp; lam[2] = -cs; lam[3] = cs; lam[4] = -cs; lam[5] = cs;
    lam[6] = lam[7] = lam[8] = R(0);
  }
  template <class R>
  __device__ static void ncp(const R* Q, const R* g, R* B) {
    const R rho = Q[9], cp = Q[10], cs = Q[11];
    const R mu = rho * cs * cs, lam = rho * cp * cp - R(2) * mu;
    R gv[3][3];  // d v_i / d x_d
    for (int i = 0; i < 3; ++i)
      for (int d = 0; d < 3; ++d) gv[i][d] = g[d * 9 + 6 + i] / rho;
    const R div = gv[0][0] + gv[1][1] + gv[2][2];
    B[0] = R(2) * mu * gv[0][0] + lam * div;
    B[1] = R(2) * mu * gv[1][1] + lam * div;
    B[2] = R(2) * mu * gv[2][2] + lam * div;
    B[3] = mu * (gv[0][1] + gv[1][0]);
    B[4] = mu * (gv[0][2] + gv[2][0]);
    B[5] = mu * (gv[1][2] + gv[2][1]);
    B[6] = B[7] = B[8] = R(0);
  }
  template <class R>
  __device__ static bool admissible(const R*) { return true; }
};
"""

ADVECTION2 = r"""
struct AdgUserPDE {
  static constexpr int DIM = 2, NV = 1, NP = 0;
  static constexpr bool LINEAR = true, HAS_NCP = false, HAS_SOURCE = true;
  template <class R>
  __device__ static void flux(const R* Q, int d, R* F) { F[0] = (d == 0 ? R(0.7) : R(-0.4)) * Q[0]; }
  template <class R>
  __device__ static void eigenvalues(const R*, int d, R* lam) { lam[0] = d == 0 ? R(0.7) : R(-0.4); }
  template <class R>
  __device__ static void source(const R* Q, R* S) { S[0] = -R(0.3) * Q[0]; }
  template <class R>
  __device__ static bool admissible(const R*) { return true; }
};
"""


def say(*a):
    print("[gpu-test]", *a, flush=True)


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


def run(s, Q0, params, steps):
    Q = dev(Q0)
    prm = dev(params) if params is not None else None
    clock = dev([0.0, 0.0])
    s.stable_dt(Q, prm, clock)
    for _ in range(steps):
        s.step(Q, prm, clock)
    torch.cuda.synchronize()
    return Q.cpu().numpy(), float(clock[0].item())


@pytest.mark.parametrize("order,cells,bc", [(3, [3, 3, 2], None), (2, [4, 2, 3], [1, 1, 0, 0, 1, 1])])
def test_user_euler_vs_oracle_and_builtin(order, cells, bc):
    say("user euler", order, cells, bc)
    P = O.problem(3, order, O.EULER, cells, bc=bc)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 81)
    su = adg.Solver(3, order, "euler", cells, source=EULER3, bc=bc)
    sb = adg.Solver(3, order, "euler", cells, bc=bc)
    assert (su.nvar, su.nparam) == (5, 0)
    Qu, tu = run(su, Q0, None, 3)
    Qb, tb = run(sb, Q0, None, 3)
    Qo, to = O.run(P, Q0, steps=3)
    say(f"  vs oracle {rel_l2(Qu, Qo):.2e}, vs built-in {rel_l2(Qu, Qb):.2e}")
    assert rel_l2(Qu, Qo) <= TOL and rel_l2(Qu, Qb) <= TOL
    assert abs(tu - to) <= 1e-14 * to
    su.close(); sb.close()


def test_user_euler_mixed_precision_matches_builtin():
    say("user euler fp32")
    cells = [3, 2, 2]
    P = O.problem(3, 3, O.EULER, cells)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 82)
    su = adg.Solver(3, 3, "euler", cells, source=EULER3, precision="fp32")
    sb = adg.Solver(3, 3, "euler", cells, precision="fp32")
    Qu, _ = run(su, Q0, None, 2)
    Qb, _ = run(sb, Q0, None, 2)
    Qo, _ = O.run(P, Q0, steps=2)
    say(f"  vs built-in fp32 {rel_l2(Qu, Qb):.2e}, vs oracle {rel_l2(Qu, Qo):.2e}")
    assert rel_l2(Qu, Qb) <= 1e-6 and rel_l2(Qu, Qo) <= 1e-5
    su.close(); sb.close()


@pytest.mark.parametrize("order,cells", [(2, [3, 2, 2]), (3, [2, 3, 2])])
def test_user_elasticity_vs_oracle(order, cells):
    say("user elastic", order, cells)
    hi = [500.0 * c for c in cells]
    P = O.problem(3, order, O.ELASTIC, cells, [0.0] * 3, hi)
    rng = np.random.default_rng(83 + order)
    params = np.column_stack([rng.uniform(2000, 3000, P.ncells), rng.uniform(5000, 7000, P.ncells),
                              rng.uniform(2500, 3400, P.ncells)])
    Q0 = inputs.elastic_smooth_state(O.node_coords(P), 84)
    s = adg.Solver(3, order, "elastic", cells, [0.0] * 3, hi, source=ELASTIC)
    assert (s.nvar, s.nparam) == (9, 3)
    Qu, _ = run(s, Q0, params, 3)
    Qo, _ = O.run(P, Q0, params, steps=3)
    e = rel_l2(Qu, Qo)
    say(f"  vs oracle {e:.2e}")
    assert e <= TOL
    with pytest.raises(adg.AdgError) as ei:  # no adjoint for a run-time PDE
        lam = dev(np.zeros_like(Q0))
        s.step_adjoint(dev(Q0), dev(params), dev([0.0, 1e-4]), lam, dev(np.zeros_like(params)))
    assert ei.value.status == -4
    s.close()


def test_user_advection_decay_vs_oracle():
    say("user advection")
    cells = [5, 4]
    P = O.problem(2, 4, O.ADVECTION, cells, adv=(0.7, -0.4, 0.0), kappa=0.3)
    xyz = O.node_coords(P)
    Q0 = (1.0 + np.sin(2 * np.pi * xyz[..., 0]) * np.cos(2 * np.pi * xyz[..., 1]))[:, None, :]
    s = adg.Solver(2, 4, "advection", cells, source=ADVECTION2)
    Qu, _ = run(s, Q0, None, 4)
    Qo, _ = O.run(P, Q0, steps=4)
    e = rel_l2(Qu, Qo)
    say(f"  vs oracle {e:.2e}")
    assert e <= TOL
    s.close()


def test_user_admissibility():
    say("user admissible")
    cells = [3, 2, 2]
    P = O.problem(3, 2, O.EULER, cells)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 85)
    Q0[4, 0, 3] = -0.5   # negative density at one node of cell 4
    Q0[7, 4, :] = 0.01   # energy too small for a positive pressure in cell 7
    s = adg.Solver(3, 2, "euler", cells, source=EULER3)
    flags = torch.zeros(P.ncells, dtype=torch.uint8, device="cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    s.check_admissible(dev(Q0), None, flags, count)
    torch.cuda.synchronize()
    oflags, ocount = O.check_admissible(P, Q0)
    assert int(count.item()) == int(ocount) == 2
    assert np.array_equal(flags.cpu().numpy().astype(bool), np.asarray(oflags).astype(bool))
    s.close()


def test_user_pde_errors():
    say("user errors")
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, 2, "euler", [2, 2, 2], source=EULER3.replace("return Q[0] > R(0)", "return Q[0] >> R(0)"))
    assert ei.value.status == -5 and "error" in str(ei.value)
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(2, 2, "euler", [2, 2], source=EULER3)  # DIM = 3 in the struct
    assert ei.value.status == -1
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, 2, "euler", [2, 2, 2], source=EULER3, bc=[2, 2, 0, 0, 0, 0])
    assert ei.value.status == -1


# Euler with the paper's boundaryValues user function: an inflow state that
# depends on the face position and the time on the low x face, the mirror
# image (a reflecting wall) elsewhere
EULER3_BV = EULER3.replace("struct AdgUserPDE {", r"""struct AdgUserPDE {
  static constexpr bool HAS_BOUNDARY = true;
  __device__ static void boundary_values(const double* x, double t, double dt, int face, const double* Qin,
                                         const double* Fin, double* Qout, double* Fout) {
    if (face == 0) {
      const double rho = 1.1 + 2.0 * (x[0] - 0.25) + 0.5 * (t - 0.3), u = 0.5, v = 0.1, p = 1.2;
      Qout[0] = rho;
      Qout[1] = rho * u;
      Qout[2] = rho * v;
      Qout[3] = 0.0;
      Qout[4] = p / 0.4 + 0.5 * rho * (u * u + v * v);
      flux<double>(Qout, 0, Fout);
    } else {
      const int d = face / 2;
      for (int k = 0; k < 5; ++k) {
        Qout[k] = Qin[k];
        Fout[k] = -Fin[k];
      }
      Qout[1 + d] = -Qin[1 + d];
      Fout[1 + d] = Fin[1 + d];
    }
  }""", 1)


def test_user_boundary_values_vs_oracle():
    # at x = 0.25 (the low face) and t = 0.3 the user's state is the oracle's
    # prescribed inflow state; the other non-periodic faces are walls
    print("[gpu-test] user boundary_values", flush=True)
    cells, lo, hi = [3, 3, 2], [0.25, 0.0, 0.0], [1.25, 1.0, 1.0]
    rho, u, v, p = 1.1, 0.5, 0.1, 1.2
    q_in = [rho, rho * u, rho * v, 0.0, p / 0.4 + 0.5 * rho * (u * u + v * v)]
    P = O.problem(3, 3, O.EULER, cells, lo, hi, bc=[O.BC_INFLOW, O.BC_WALL, 0, 0, O.BC_WALL, O.BC_WALL],
                  bc_state={0: q_in})
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 77)
    dt = 0.5 * O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.3)
    s = adg.Solver(3, 3, "euler", cells, lo, hi, source=EULER3_BV,
                   bc=["user", "user", "periodic", "periodic", "user", "user"])
    Q = torch.as_tensor(Q0, device="cuda")
    s.step(Q, None, torch.tensor([0.3, dt], dtype=torch.float64, device="cuda"), next_dt=False)
    torch.cuda.synchronize()
    e = float(np.linalg.norm(Q.cpu().numpy() - Qo) / np.linalg.norm(Qo))
    print(f"[gpu-test]   rel L2 vs oracle {e:.2e}", flush=True)
    assert e <= TOL
    s.close()
    # without boundary_values the user face kind is refused
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, 2, "euler", cells, source=EULER3, bc=["user", "user", 0, 0, 0, 0])
    assert ei.value.status == -1
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, 2, "euler", cells, bc=["user", "user", 0, 0, 0, 0])
    assert ei.value.status == -1


@pytest.mark.parametrize("order", [2, 3])
def test_user_euler_point_source_vs_builtin(order):
    """The run-time PDE's predictor with a point source (its own kernel where
    lines are used) against the built-in Euler's."""
    cells = [3, 2, 3]
    src = dict(x=[0.4, 0.3, 0.7], weight=[0.0, 0.1, 0.2, -0.1, 0.4], f0=2.0, t0=0.1, amp=0.02)
    P = O.problem(3, order, O.EULER, cells)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 83)
    out = []
    for kw in (dict(source=EULER3), {}):
        s = adg.Solver(3, order, "euler", cells, **kw)
        s.set_point_sources([src])
        out.append(run(s, Q0, None, 2)[0])
        s.close()
    assert rel_l2(out[0], out[1]) <= TOL
    assert rel_l2(out[1], Q0) > 1e-6


@pytest.mark.parametrize("order,cells", [(5, [41, 43]), (5, [42, 43]), (6, [42, 43]), (7, [41, 43]), (7, [42, 43])])
def test_user_source_term_on_either_side_of_the_pair_rule(order, cells):
    """A run-time PDE with a source term that is not declared linear, on 2-D
    meshes just below and above the cell count up to which lane pairs take
    its predictor: advection with decay against the oracle."""
    P = O.problem(2, order, O.ADVECTION, cells, adv=(0.7, -0.4, 0.0), kappa=0.3)
    s = adg.Solver(2, order, "advection", cells, source=ADVECTION2.replace("LINEAR = true", "LINEAR = false"))
    Q0 = np.random.default_rng(90 + order).normal(size=(P.ncells, 1, P.S))
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.0)
    Q, clock = dev(Q0), dev([0.0, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    assert rel_l2(Q.cpu().numpy(), Qo) <= TOL
    s.close()


def euler_with_scalars(k):
    """Euler with k quantities more, densities carried with the flow."""
    return (EULER3.replace("NV = 5", f"NV = {5 + k}")
            .replace("F[4] = ud * (Q[4] + p);", f"F[4] = ud * (Q[4] + p); for (int i = 5; i < {5 + k}; ++i) F[i] = ud * Q[i];")
            .replace("lam[4] = u + c;", f"lam[4] = u + c; for (int i = 5; i < {5 + k}; ++i) lam[i] = u;"))


@pytest.mark.parametrize("order,extra", [(4, 0), (4, 1), (4, 3), (5, 1), (5, 2), (5, 3)])
def test_user_single_precision_with_many_quantities(order, extra):
    """The FP32 predictor at 5^3 and 6^3 nodes per cell with up to 8 quantities
    (its rows there depend on how many lines a block has threads for).  Bar:
    1e-5, that of the mixed-precision predictor, the carried densities being
    the same multiple of the density after the step."""
    say("user fp32 quantities", order, 5 + extra)
    cells = [3, 1, 3]
    P = O.problem(3, order, O.EULER, cells)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 91)
    f = 0.5 + 0.7 * np.arange(extra)
    s = adg.Solver(3, order, "euler", cells, source=euler_with_scalars(extra), precision="fp32")
    Qu, _ = run(s, np.concatenate([Q0, Q0[:, :1] * f[None, :, None]], axis=1), None, 2)
    Qo, _ = O.run(P, Q0, steps=2)
    assert rel_l2(Qu[:, :5], Qo) <= 1e-5
    for i in range(extra):
        assert rel_l2(Qu[:, 5 + i], f[i] * Qo[:, 0]) <= 1e-5
    # every cell's increment, not only the mean: no cell took another's rows
    assert np.abs(Qu[:, :5] - Qo).max() <= 1e-4 * np.abs(Qo - Q0).max()
    s.close()


@pytest.mark.parametrize("change", [("DIM = 3", "DIM = 4"), ("NV = 5", "NV = 0"), ("NP = 0", "NP = -1"),
                                    ("NP = 0", "NP = 12")])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_user_sizes_are_an_invalid_argument(change, precision):
    # the struct's sizes are looked at before anything is compiled for them
    say("user sizes", change, precision)
    with pytest.raises(adg.AdgError) as ei:
        adg.Solver(3, 3, "euler", [3, 2, 2], source=EULER3.replace(*change), precision=precision)
    assert ei.value.status == -1 and "AdgUserPDE" in str(ei.value)
