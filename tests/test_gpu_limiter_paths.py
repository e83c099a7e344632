"""The limited step's kernels where their work split changes (through the
C ABI): 2-D cells packed several to a wave (every order the limiter is built
for, cell counts that leave a wave part full), and meshes large enough for
one wave to look through several cells.

Bars: those of the limiter's oracle tests (statuses and counts exact, state
and FV subcells 1e-12 relative L2, the time step 1e-12 relative); a run that
reuses its subcell ranges is bitwise the run that projects every cell.
"""
import numpy as np
import pytest

import oracle as O
from test_gpu_limiter import OUT, PER, W, blast_case, dev, rel_l2, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,order,cells,bc", [
    (2, 1, [11, 7], [W] * 4),             # 8 cells per wave, 77 cells
    (2, 4, [9, 5], [W, OUT, PER, PER]),   # 7 per wave
    (2, 6, [6, 5], [W] * 4),              # 4 per wave
    (2, 7, [5, 5], [OUT, W, W, W]),       # 4 per wave
    (2, 7, [1, 3], [PER, PER, W, W]),     # fewer cells than one wave holds
    (3, 1, [5, 1, 7], [W, W, PER, PER, OUT, W]),
])
def test_every_split_matches_the_oracle(dim, order, cells, bc):
    say("limiter split", dim, order, cells)
    P, s, Q, sub, st = blast_case(dim, order, cells, bc, seed=7, radius=0.3)
    dt = 0.5 * O.stable_dt(P, Q)[0]
    Qg, sin, stg = dev(Q), dev(sub), dev(st, torch.uint8)
    sout = torch.zeros_like(sin)
    counts = torch.zeros(3, dtype=torch.int32, device="cuda")
    Qo, subo, sto = Q, sub, st
    t = 0.0
    clock = dev([0.0, dt])
    for k in range(2):
        Qo, subo, sto, co = O.step_limited(P, Qo, dt, t, sub=subo, status=sto)
        s.step_limited(Qg, clock, sin, sout, stg, counts, next_dt=True, reuse_ranges=True)
        torch.cuda.synchronize()
        sin, sout = sout, sin
        t1, dt1 = s.read_clock(clock)
        dto = O.stable_dt_limited(P, Qo, subo, sto)[0]
        fv = sto >= 2
        e_q = rel_l2(Qg.cpu().numpy(), Qo)
        e_s = rel_l2(sin.cpu().numpy()[fv], subo[fv]) if fv.any() else 0.0
        say(f"  step {k}: counts {co}, state {e_q:.2e}, subcells {e_s:.2e}, dt {dt1 / dto - 1:.1e}")
        assert np.array_equal(stg.cpu().numpy(), sto) and tuple(counts.cpu().numpy()) == co
        assert e_q <= 1e-12 and e_s <= 1e-12 and abs(dt1 - dto) <= 1e-12 * dto
        t += dt
        dt = 0.5 * dt  # (not the GPU's own: both sides step alike)
        clock = dev([t, dt])
    s.close()


@pytest.mark.parametrize("dim,cells", [(2, [210, 171]), (3, [37, 36, 35])])
def test_several_cells_per_wave(dim, cells):
    # 2 cells per wave from 32768 cells: ranges left in place, speeds of
    # untouched cells taken from the corrector
    say("limiter cells per wave", dim, cells)
    P, s, Q, sub, st = blast_case(dim, 1, cells, [W] * (2 * dim), seed=3, radius=0.3)
    runs = []
    for reuse in (False, True):
        Qg, sin, stg = dev(Q), dev(sub), dev(st, torch.uint8)
        sout = torch.zeros_like(sin)
        counts = torch.zeros(3, dtype=torch.int32, device="cuda")
        clock = torch.zeros(2, dtype=torch.float64, device="cuda")
        s.stable_dt(Qg, None, clock)
        hist = []
        for _ in range(4):
            s.step_limited(Qg, clock, sin, sout, stg, counts, next_dt=True, reuse_ranges=reuse)
            sin, sout = sout, sin
            fvm = stg >= 2
            hist.append((Qg.clone(), stg.clone(), torch.where(fvm[:, None, None], sin, 0.0), counts.clone(),
                         clock.clone()))
        torch.cuda.synchronize()
        runs.append(hist)
    for k, (a, b) in enumerate(zip(*runs)):
        assert all(torch.equal(x, y) for x, y in zip(a, b)), f"step {k}"
    Qh, sth, subh, ch, clk = (x.cpu().numpy() for x in runs[1][-1])
    dto = O.stable_dt_limited(P, Qh, subh, sth)[0]
    # the solver's own Courant number (the problem's is O's)
    ratio = O.stable_dt(P, Q)[0] / float(_dt0(s, Q))
    say(f"  counts {tuple(ch)}, dt {clk[1] * ratio / dto - 1:.1e}")
    assert ch[1] > 0 and ch[2] > 0
    assert abs(clk[1] * ratio - dto) <= 1e-12 * dto
    s.close()


def test_captured_limited_steps_replay():
    """Two limited steps that reuse their ranges, captured and replayed with
    eager work between the replays: bitwise the run launched step by step
    (which of the two range arrays is current is kept on the device)."""
    P, s, Q, sub, st = blast_case(2, 3, [24, 20], [W] * 4, seed=13, radius=0.3)
    out = []
    for captured in (False, True):
        Qg, a, stg = dev(Q), dev(sub), dev(st, torch.uint8)
        b = torch.zeros_like(a)
        counts = torch.zeros(3, dtype=torch.int32, device="cuda")
        clock = torch.zeros(2, dtype=torch.float64, device="cuda")
        s.stable_dt(Qg, None, clock)
        kw = dict(next_dt=True, reuse_ranges=True)
        s.step_limited(Qg, clock, a, b, stg, counts)  # (a new state: nothing to reuse)
        s.step_limited(Qg, clock, b, a, stg, counts, **kw)
        torch.cuda.synchronize()

        def pair(stream=None):
            s.step_limited(Qg, clock, a, b, stg, counts, stream=stream, **kw)
            s.step_limited(Qg, clock, b, a, stg, counts, stream=stream, **kw)

        hist = []
        if captured:
            side = torch.cuda.Stream()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                pair(side.cuda_stream)
        for _ in range(4):
            graph.replay() if captured else pair()
            torch.cuda.synchronize()
            hist.append((Qg.clone(), stg.clone(), counts.clone(), clock.clone()))
            float(Qg.sum())  # eager work between the replays
        out.append(hist)
    for x, y in zip(*out):
        assert all(torch.equal(p, q) for p, q in zip(x, y))
    assert int(out[1][-1][2][1]) > 0
    s.close()


def _dt0(s, Q):
    clock = torch.zeros(2, dtype=torch.float64, device="cuda")
    s.stable_dt(dev(Q), None, clock)
    torch.cuda.synchronize()
    return s.read_clock(clock)[1]


@pytest.mark.parametrize("order,cells", [(5, [49, 40]), (5, [50, 41]), (7, [45, 45])])
def test_packed_detection_at_high_order(order, cells):
    # either side of the cell count from which 2-D cells of N >= 5 share a wave
    test_every_split_matches_the_oracle(2, order, cells, [W] * 4)
