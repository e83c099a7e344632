"""The FP64 predictor's geometries where they can go wrong.  One lane per line
(3-D Euler, N <= 3): one cell, ragged last waves, sources on and off, one and
two Picard passes (N = 3 takes the other kernel there), the CERK guess; and a
NaN node, which stays in its own cell's results.  2-D meshes on either side
of the cell counts from which lines (N = 2, 3) and packed blocks (N = 4, 5, 6)
are used.

Bar: relative L2 <= 1e-12 against the oracle's step (the predictor's sums are
reordered, each value is a few hundred FP64 operations: about 1e-14).
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


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("order", [1, 2, 3])
@pytest.mark.parametrize("cells", [[1, 1, 1], [3, 5, 2], [4, 4, 5]])
@pytest.mark.parametrize("iters,guess,source", [(0, "constant", False), (0, "constant", True), (1, "constant", False),
                                                (2, "constant", True), (3, "cerk", False), (0, "cerk", True)])
def test_step_against_oracle(order, cells, iters, guess, source):
    print("[gpu-test] line predictor", order, cells, iters, guess, source, flush=True)
    src = dict(x=[0.3, 0.45, 0.55], weight=[0.0, 0.2, -0.1, 0.3, 0.5], w=[0.0, 0.2, -0.1, 0.3, 0.5], f0=2.0, t0=0.1,
               amp=0.05)
    kw = dict(cfl=0.4, picard_iters=iters or None)
    P = O.problem(3, order, O.EULER, cells, sources=[src] if source else (),
                  guess=O.GUESS_CERK if guess == "cerk" else 0, **kw)
    s = adg.Solver(3, order, "euler", cells, cfl=0.4, picard_iters=iters, initial_guess=guess)
    if source:
        s.set_point_sources([src])
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 17)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.05)
    Q, clock = dev(Q0), dev([0.05, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    assert rel_l2(Q.cpu().numpy(), Qo) <= TOL
    s.close()


@pytest.mark.parametrize("order,cells", [(2, [125, 119]), (2, [125, 121]), (3, [131, 117]), (4, [70, 71]), (4, [73, 71]),
                                         (5, [71, 73]), (6, [67, 79])])
@pytest.mark.parametrize("guess,source", [("constant", False), ("constant", True), ("cerk", False)])
def test_step_2d_against_oracle(order, cells, guess, source):
    print("[gpu-test] 2-D predictor", order, cells, guess, source, flush=True)
    src = dict(x=[0.98, 0.97], weight=[0.0, 0.2, -0.1, 0.5], w=[0.0, 0.2, -0.1, 0.5], f0=2.0, t0=0.1, amp=1e-3)
    P = O.problem(2, order, O.EULER, cells, cfl=0.4, sources=[src] if source else (),
                  guess=O.GUESS_CERK if guess == "cerk" else 0)
    s = adg.Solver(2, order, "euler", cells, cfl=0.4, initial_guess=guess)
    if source:
        s.set_point_sources([src])
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 19)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.05)
    Q, clock = dev(Q0), dev([0.05, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    assert rel_l2(Q.cpu().numpy(), Qo) <= TOL
    last = P.ncells - 1  # the cell with the source, in the last block
    assert rel_l2(Q[last].cpu().numpy(), Qo[last]) <= TOL
    s.close()


@pytest.mark.parametrize("order,cells", [(5, [54, 55]), (5, [55, 56]), (7, [27, 28]), (7, [28, 28])])
def test_small_mesh_rules_against_oracle(order, cells):
    # either side of the counts for lane pairs (N = 7, which have no CERK guess)
    # and packed blocks (N = 5)
    test_step_2d_against_oracle(order, cells, "constant", True)
    test_step_2d_against_oracle(order, cells, "cerk", False)


@pytest.mark.parametrize("cells", [[1, 1, 1], [3, 5, 2], [7, 8, 7], [9, 9, 8]])
@pytest.mark.parametrize("iters,guess,source", [(0, "constant", True), (1, "constant", False), (0, "cerk", False)])
def test_five_cubed_rows_against_oracle(cells, iters, guess, source):
    # 3-D N = 4: slice pairs, lane pairs, and the rows laid out a direction at a
    # time, by the number of cells
    test_step_against_oracle(4, cells, iters, guess, source)


@pytest.mark.parametrize("iters,guess,source", [(0, "constant", False), (0, "constant", True), (2, "constant", True),
                                                (3, "cerk", False), (0, "cerk", True)])
def test_matrix_lines_against_oracle(iters, guess, source):
    # 3-D N = 3 at a cell count that takes lines, the last wave part full
    test_step_against_oracle(3, [9, 9, 9], iters, guess, source)


@pytest.mark.parametrize("dim,order,cells", [(2, 1, [5, 7]), (2, 4, [7, 3]), (2, 6, [3, 5]), (2, 7, [3, 3]), (3, 2, [3, 2, 5]),
                                             (3, 4, [1, 1, 1]), (3, 4, [3, 1, 3]), (3, 5, [1, 2, 1])])
def test_fp32_rows_against_oracle(dim, order, cells):
    """The FP32 predictor's LDS rows at ragged cell counts; bar: 1e-5, that of
    the mixed-precision predictor against the FP64 oracle."""
    print("[gpu-test] fp32 rows", dim, order, cells, flush=True)
    P = O.problem(dim, order, O.EULER, cells, cfl=0.4)
    s = adg.Solver(dim, order, "euler", cells, cfl=0.4, precision="fp32")
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 29)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.0)
    Q, clock = dev(Q0), dev([0.0, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    g = Q.cpu().numpy()
    assert rel_l2(g, Qo) <= 1e-5
    # every cell's increment, not only the mean: no cell took another's rows
    assert np.abs(g - Qo).max() <= 1e-4 * np.abs(Qo - Q0).max()
    s.close()


@pytest.mark.parametrize("order,cells", [(1, [4, 3, 3]), (2, [4, 3, 3]), (3, [4, 3, 3]), (3, [9, 9, 9])])
def test_nan_stays_in_its_cell(order, cells):
    s = adg.Solver(3, order, "euler", cells, cfl=0.4)
    P = O.problem(3, order, O.EULER, cells, cfl=0.4)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 23)
    dt = O.stable_dt(P, Q0)[0]
    ref = torch.empty(s.state_shape, dtype=torch.float64, device="cuda")
    s.predict(dev(Q0), None, dev([0.0, dt]), ref)
    bad = Q0.copy()
    bad[13, 0, 1] = np.nan
    out, tr = torch.empty_like(ref), torch.empty(s.trace_shape, dtype=torch.float64, device="cuda")
    s.predict(dev(bad), None, dev([0.0, dt]), out, tr)
    torch.cuda.synchronize()
    keep = np.arange(P.ncells) != 13
    assert torch.equal(out[keep], ref[keep]) and bool(torch.isfinite(tr[keep]).all())
    assert bool(torch.isnan(out[13, 0]).any())
    s.close()


@pytest.mark.parametrize("order,cells,iters,guess,source", [
    (2, [19, 14, 15], 0, "cerk", False), (2, [20, 20, 10], 0, "cerk", False),
    (2, [17, 31, 11], 0, "cerk", True), (2, [20, 29, 10], 0, "cerk", True),
    (3, [10, 17, 7], 0, "cerk", False), (3, [10, 12, 10], 0, "cerk", False),
    (3, [9, 13, 17], 0, "cerk", True), (3, [10, 20, 10], 0, "cerk", True),
    (4, [8, 8, 8], 1, "constant", False), (4, [8, 8, 8], 2, "constant", True), (4, [3, 9, 19], 2, "constant", True)])
def test_three_dimensional_rules_against_oracle(order, cells, iters, guess, source):
    # either side of the cell counts and passes for lines (N = 2, 3 with the
    # CERK guess) and lane pairs (N = 4)
    test_step_against_oracle(order, cells, iters, guess, source)


@pytest.mark.parametrize("order,cells,iters", [(7, [16, 32], 4), (7, [16, 32], 5), (7, [19, 27], 5), (2, [125, 120], 1),
                                               (2, [125, 120], 2), (3, [125, 120], 1)])
def test_two_dimensional_rules_against_oracle(order, cells, iters):
    # either side of the cells and passes for lane pairs and for lines
    print("[gpu-test] 2-D rules", order, cells, iters, flush=True)
    P = O.problem(2, order, O.EULER, cells, cfl=0.4, picard_iters=iters)
    s = adg.Solver(2, order, "euler", cells, cfl=0.4, picard_iters=iters)
    Q0 = inputs.smooth_euler_state(O.node_coords(P), 31)
    dt = O.stable_dt(P, Q0)[0]
    Qo = O.step(P, Q0, None, dt, 0.0)
    Q, clock = dev(Q0), dev([0.0, dt])
    s.step(Q, None, clock, next_dt=False)
    torch.cuda.synchronize()
    assert rel_l2(Q.cpu().numpy(), Qo) <= TOL
    s.close()


@pytest.mark.parametrize("order,tiles", [(2, [12, 12]), (3, [31, 30]), (4, [9, 9]), (5, [9, 9]), (6, [9, 9]), (7, [9, 9])])
def test_fp32_single_accesses_are_the_paired_ones_bitwise(order, tiles):
    """2-D meshes on which the FP32 predictor accesses its rows one element at
    a time: a periodic mesh of 13 x 17 cells, repeated until it has as many
    cells, steps bitwise as the small one, whose rows are accessed in pairs
    (itself against the oracle, 1e-5).  The last block is part full."""
    print("[gpu-test] fp32 single accesses", order, tiles, flush=True)
    small, h = [13, 17], 1.0 / 16
    P = O.problem(2, order, O.EULER, small, [0.0, 0.0], [n * h for n in small], cfl=0.4)
    x = O.node_coords(P) * (1.0 / np.array([n * h for n in small]))
    Q0 = inputs.smooth_euler_state(x, 37)
    dt = O.stable_dt(P, Q0)[0]
    out = []
    for t in ([1, 1], tiles):
        cells = [n * k for n, k in zip(small, t)]
        s = adg.Solver(2, order, "euler", cells, [0.0, 0.0], [n * h for n in cells], cfl=0.4, precision="fp32")
        Q = dev(np.tile(Q0.reshape(small[1], small[0], 4, -1), (t[1], t[0], 1, 1)).reshape(s.state_shape))
        s.step(Q, None, dev([0.0, dt]), next_dt=False)
        torch.cuda.synchronize()
        out.append(Q.view(t[1], small[1], t[0], small[0], 4, -1))
        s.close()
    assert rel_l2(out[0].cpu().numpy().reshape(Q0.shape), O.step(P, Q0, None, dt, 0.0)) <= 1e-5
    assert torch.equal(out[1], out[0].expand_as(out[1]))
