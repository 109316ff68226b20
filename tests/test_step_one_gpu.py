"""The IB pass in arcs and the one-launch step, through the C ABI: against the
FP64 oracle where the number of arcs changes, and one-launch steps bit for bit
against plain steps (the same passes in launches of their own) where the pass
waits for faces, closes walls itself or follows a fast body."""
import numpy as np
import pytest

import ib_cases
import oracle
import paper_2609_02298_amd as ib
from paper_2609_02298_amd import ib_lbm

pytestmark = pytest.mark.gpu

# velocity and populations, relative to their maximum (double precision)
F64_FIELD, F64_DRAG = 1e-12, 1e-10


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    ib.load_library()


def rel(a, b):
    return float(np.abs(np.asarray(a) - np.asarray(b)).max() / max(np.abs(b).max(), 1e-300))


def box(nx, ny, bodies, bc, col=ib.TRT, **kw):
    return dict(nx=nx, ny=ny, collision=col, tau=0.68, trt_magic=0.25, cm_s_q=1.2, cm_s_eps=1.4, bc=bc,
                bodies=bodies, **kw)


FAR = (ib.VEL_UNIFORM, ib.ZERO_GRADIENT, ib.VEL_UNIFORM, ib.VEL_UNIFORM)


# markers per workgroup: 64 (P4) or 128 (hat) at 256 threads, FP32 DFC in one arc
# up to 512 threads (P4), MDF of five passes up to 1024; below, at and above each bound, and many arcs
@pytest.mark.parametrize("scheme,kernel,nb", [
    (ib.DF, ib.PESKIN4, 64), (ib.DF, ib.PESKIN4, 65), (ib.DF, ib.PESKIN4, 301),
    (ib.DF, ib.HAT, 128), (ib.DF, ib.HAT, 129), (ib.DF, ib.HAT, 301),
    (ib.DFC, ib.PESKIN4, 64), (ib.DFC, ib.PESKIN4, 65), (ib.DFC, ib.PESKIN4, 128),
    (ib.DFC, ib.PESKIN4, 129), (ib.DFC, ib.PESKIN4, 200),
    (ib.DFC, ib.HAT, 128), (ib.DFC, ib.HAT, 129), (ib.DFC, ib.HAT, 301),
    (ib.MDF, ib.PESKIN4, 64), (ib.MDF, ib.PESKIN4, 65), (ib.MDF, ib.PESKIN4, 128),
    (ib.MDF, ib.PESKIN4, 129), (ib.MDF, ib.PESKIN4, 301),
    (ib.MDF, ib.HAT, 128), (ib.MDF, ib.HAT, 129), (ib.MDF, ib.HAT, 301)])
def test_arcs_match_the_oracle(scheme, kernel, nb):
    D = nb / np.pi
    n = int(D) + 40
    print(f"arcs scheme={scheme} kernel={kernel} markers={nb}", flush=True)
    case = box(n + 30, n, [dict(xc=n / 2 + 0.37, yc=n / 2 - 0.21, diameter=D, n_markers=nb, scheme=scheme,
                                kernel=kernel, mdf_iters=5)], FAR, u_bc=0.06)
    for over in (False, True):
        sim, ref = ib.Sim(case), oracle.OracleSim(case)
        sim.set_overlap(over)
        ref.add_body(case["bodies"][0])
        for k in (1, 7):
            sim.step(k)
            ref.step(k)
            assert sim.step_form() == (ib.STEP_ONE if over and k > 1 else ib.STEP_PLAIN)
            a, b = sim.forces(0), ref.body_state(0)
            assert abs(a["fx"] - b["fx"]) < F64_DRAG * abs(b["fx"])
            assert abs(a["torque"] - b["torque"]) < F64_DRAG * abs(b["fx"]) * D
            assert abs(a["slip_mean"] - b["slip_mean"]) < 1e-10 * max(b["slip_mean"], 1e-12)
        assert rel(sim.populations(), ref.populations()) < F64_FIELD
        sim.close()
        ref.close()


# FP32: strips by columns (Peskin) and rows, DFC in one arc up to 128 markers.  A
# population's rounding (2^-24 of at most its maximum) enters each of the eight
# steps through its nine-term sums
@pytest.mark.parametrize("scheme,kernel,nb", [
    (ib.DFC, ib.PESKIN4, 64), (ib.DFC, ib.PESKIN4, 65), (ib.DFC, ib.PESKIN4, 128), (ib.DFC, ib.PESKIN4, 129),
    (ib.DFC, ib.HAT, 129), (ib.DF, ib.PESKIN4, 65), (ib.DF, ib.HAT, 129), (ib.MDF, ib.PESKIN4, 129),
    (ib.MDF, ib.HAT, 301)])
def test_fp32_arcs_match_the_oracle(scheme, kernel, nb):
    D = nb / np.pi
    n = int(D) + 40
    print(f"fp32 arcs scheme={scheme} kernel={kernel} markers={nb}", flush=True)
    case = box(n + 30, n, [dict(xc=n / 2 + 0.37, yc=n / 2 - 0.21, diameter=D, n_markers=nb, scheme=scheme,
                                kernel=kernel, mdf_iters=5)], FAR, u_bc=0.06)
    sim, ref = ib.Sim(case, precision=ib.FP32_SHIFTED), oracle.OracleSim(case)
    ref.add_body(case["bodies"][0])
    sim.step(8)
    ref.step(8)
    assert sim.step_form() == ib.STEP_ONE
    a, b = sim.forces(0), ref.body_state(0)
    bound = 8 * 9 * 2.0 ** -24
    assert rel(sim.populations(), ref.populations()) < bound
    # a marker's force is a difference of populations of at least 1/20 of them
    assert abs(a["fx"] - b["fx"]) < 20 * bound * abs(b["fx"])
    sim.close()
    ref.close()


# marker spacings just below and above those at which one neighbour more shares
# a support node (ns sqrt 2 / j), where the band half-width steps
@pytest.mark.parametrize("side", [0.97, 1.03])
@pytest.mark.parametrize("scheme", [ib.DF, ib.MDF, ib.DFC])
@pytest.mark.parametrize("kernel,j", [(ib.HAT, 2), (ib.HAT, 3), (ib.PESKIN4, 5), (ib.PESKIN4, 6)])
def test_band_width_at_its_steps(kernel, j, scheme, side):
    nb = 180
    D = nb * side * (2 if kernel == ib.HAT else 4) * 2 ** 0.5 / j / np.pi
    n = int(D) + 40
    print(f"band scheme={scheme} kernel={kernel} neighbours={j} side={side}", flush=True)
    case = box(n + 30, n, [dict(xc=n / 2 + 0.37, yc=n / 2 - 0.21, diameter=D, n_markers=nb, scheme=scheme,
                                kernel=kernel, mdf_iters=3)], FAR, u_bc=0.06)
    sim, ref = ib.Sim(case), oracle.OracleSim(case)
    ref.add_body(case["bodies"][0])
    sim.step(6)
    ref.step(6)
    a, b = sim.forces(0), ref.body_state(0)
    assert abs(a["fx"] - b["fx"]) < F64_DRAG * abs(b["fx"])
    assert rel(sim.populations(), ref.populations()) < F64_FIELD
    sim.close()
    ref.close()


def free(x, y, D, scheme, kernel, **kw):
    return dict(xc=x, yc=y, diameter=D, scheme=scheme, kernel=kernel, mdf_iters=3, motion=ib.FREE,
                density_ratio=1.6, internal_mass=ib.IM_FENG, **kw)


ZOU = (ib.ZOU_HE,) * 4
PER = (ib.PERIODIC,) * 4
CASES = {
    # supports on the wall nodes of a corner: the pass waits for the faces and
    # closes the walls it reads
    "corner-DF": box(60, 50, [free(7.3, 7.6, 12.0, ib.DF, ib.PESKIN4)], ZOU, gravity=(2e-5, 3e-5)),
    "corner-DFC": box(60, 50, [free(51.6, 41.6, 12.0, ib.DFC, ib.PESKIN4)], ZOU, ib.CMMRT,
                      gravity=(-1e-5, -2e-5)),
    "wall-MDF": box(60, 50, [free(30.2, 7.4, 12.0, ib.MDF, ib.HAT)], (ib.PERIODIC, ib.PERIODIC, ib.ZOU_HE,
                                                                       ib.ZOU_HE), gravity=(2e-5, 1e-5)),
    "wall-DFC": box(60, 50, [free(30.2, 43.1, 11.0, ib.DFC, ib.HAT)], (ib.PERIODIC, ib.PERIODIC, ib.ZOU_HE,
                                                                        ib.ZOU_HE), gravity=(2e-5, 0.0)),
    # supports on the seam of a periodic lattice, and on open faces
    "seam-DF": box(70, 66, [free(8.2, 33.3, 13.0, ib.DF, ib.PESKIN4)], PER, ib.BGK, gravity=(0.0, 2e-5)),
    "open-MDF": box(70, 66, [free(60.9, 57.3, 13.0, ib.MDF, ib.PESKIN4)], (ib.ZERO_GRADIENT,) * 4,
                    gravity=(-2e-5, -2e-5)),
    # two bodies, one above the other, until their supports could meet
    "meet-DF": box(80, 120, [free(40.0, 70.0, 14.0, ib.DF, ib.HAT),
                             free(41.0, 93.0, 14.0, ib.DF, ib.HAT, amp=(0.0, 0.0))], (ib.BOUNCE_BACK,) * 4,
                   gravity=(0.0, -4e-4)),
    # a driven body that crosses several nodes per step (hardly relaxed, so
    # that the flow stays subsonic), and a slower one
    "fast-MDF": box(200, 90, [dict(xc=90.0, yc=45.3, diameter=14.0, scheme=ib.MDF, kernel=ib.PESKIN4,
                                   mdf_iters=4, mdf_omega=1e-3, motion=ib.PRESCRIBED_SIN, amp=(40.0, 6.0),
                                   freq=0.02, phase=0.4)], FAR, u_bc=0.02),
    "driven-DFC": box(200, 90, [dict(xc=90.0, yc=45.3, diameter=14.0, scheme=ib.DFC, kernel=ib.HAT,
                                   motion=ib.PRESCRIBED_SIN, amp=(20.0, 0.0), freq=0.002, phase=0.4)],
                    FAR, ib.CMMRT, u_bc=0.02),
    # moving bodies of several arcs (more than 64 markers at the Peskin kernel,
    # 128 for DFC): in the open, on a wall and in a corner that the arcs close
    # themselves, and driven
    "arcs-DFC": box(120, 110, [free(60.3, 50.6, 46.0, ib.DFC, ib.PESKIN4)], PER, ib.CMMRT,
                    gravity=(1e-5, 2e-5)),
    "wall-arcs-DFC": box(120, 90, [free(60.3, 24.4, 46.0, ib.DFC, ib.PESKIN4)], ZOU, ib.CMMRT,
                         gravity=(2e-5, 1e-6)),
    "corner-arcs-DFC": box(120, 90, [free(94.6, 64.6, 46.0, ib.DFC, ib.PESKIN4)], ZOU, ib.TRT,
                           gravity=(-1e-6, -2e-6)),
    "corner-arcs-DF": box(120, 90, [free(16.4, 72.6, 30.0, ib.DF, ib.PESKIN4)], ZOU, ib.TRT,
                          gravity=(1e-6, -2e-6)),
    "pair-arcs-DFC": box(130, 170, [free(60.3, 40.6, 46.0, ib.DFC, ib.PESKIN4),
                                    free(66.1, 114.2, 56.0, ib.DFC, ib.PESKIN4)], (ib.BOUNCE_BACK,) * 4, ib.BGK,
                         gravity=(0.0, -2e-5)),
    "driven-arcs-DF": box(260, 160, [dict(xc=100.0, yc=80.3, diameter=80.0, scheme=ib.DF, kernel=ib.PESKIN4,
                                          motion=ib.PRESCRIBED_SIN, amp=(0.0, 12.0), freq=0.002, phase=0.4)],
                          FAR, ib.CMMRT, u_bc=0.03),
    "driven-arcs-MDF": box(300, 190, [dict(xc=120.0, yc=95.3, diameter=100.0, scheme=ib.MDF, kernel=ib.PESKIN4,
                                           mdf_iters=3, motion=ib.PRESCRIBED_SIN, amp=(15.0, 5.0), freq=0.002,
                                           phase=0.4)], FAR, u_bc=0.03),
    # no body: tiles and faces alone
    "empty-open": box(131, 47, [], (ib.ZERO_GRADIENT,) * 4, ib.CMMRT),
    "empty-3x3": box(3, 3, [], PER),
    "empty-5x4": box(5, 4, [], (ib.BOUNCE_BACK,) * 4, ib.BGK),
    "empty-box": box(64, 33, [], ZOU, ib.BGK, fluid_force=(1e-6, -2e-6)),
}


def plain_and_one_launch(case, prec, calls):
    """What plain steps, one-launch steps and replayed one-launch steps leave
    after each call."""
    pops = ib_cases.random_populations(case["nx"], case["ny"], 5, amp=0.004, u=(0.01, 0.005))
    runs = []
    for over, graph in ((False, 0), (True, 0), (True, 6)):
        sim = ib.Sim(case, precision=prec)
        sim.set_overlap(over)
        sim.set_populations(pops)
        sim.set_graph(graph)
        seen = []
        for k in calls:
            sim.step(k)
            assert sim.step_form() == (ib.STEP_ONE if over and (k > 1 or seen) else ib.STEP_PLAIN)
            st = [sim.forces(b, check=False) for b in range(len(case["bodies"]))]
            seen.append((sim.steps_done, sim.populations(), sim.force(), st))
        runs.append(seen)
        sim.close()
    return runs


def assert_same(runs):
    for seen in runs[1:]:
        for (n0, p0, f0, s0), (n1, p1, f1, s1) in zip(runs[0], seen):
            assert n0 == n1 and np.isfinite(p0).all()
            assert np.array_equal(p0, p1)
            assert np.array_equal(f0[0], f1[0]) and np.array_equal(f0[1], f1[1])
            assert s0 == s1


@pytest.mark.parametrize("prec", [ib.FP64, ib.FP32_SHIFTED])
@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_steps_are_bitwise_the_plain_steps(name, prec):
    print(f"one-launch {name} prec={prec}", flush=True)
    assert_same(plain_and_one_launch(CASES[name], prec, (1, 2, 13, 24)))


# DFC bodies that correct nodes of a Zou-He wall until the case halts: the
# support leaves the lattice, or the body becomes too fast ("slide").  The step
# that fails is not completed, and the lattice it started from is read back.
# One arc and several; on a wall and in a corner
HALTS = {
    "fall-P4": (14.0, ib.PESKIN4, (30.2, 8.4), (0.0, -8e-3), "E_RANGE"),
    "fall-hat": (14.0, ib.HAT, (30.2, 7.5), (0.0, -8e-3), "E_RANGE"),
    "fall-P4-arcs": (46.0, ib.PESKIN4, (30.2, 24.4), (0.0, -8e-3), "E_RANGE"),
    "corner-P4-arcs": (46.0, ib.PESKIN4, (34.6, 24.4), (6e-3, -6e-3), "E_RANGE"),
    "slide-P4": (14.0, ib.PESKIN4, (22.2, 8.4), (0.3, 0.0), "E_DIVERGED"),
    "slide-hat-arcs": (42.0, ib.HAT, (24.2, 21.5), (0.3, 0.0), "E_DIVERGED"),
}


@pytest.mark.parametrize("prec", [ib.FP64, ib.FP32_SHIFTED])
@pytest.mark.parametrize("name", list(HALTS))
def test_a_case_halted_at_a_wall_is_left_as_plain_steps_leave_it(name, prec):
    D, kernel, (x, y), g, status = HALTS[name]
    print(f"halt at a wall {name} prec={prec}", flush=True)
    case = box(60, 60, [free(x, y, D, ib.DFC, kernel)], ZOU, ib.CMMRT, gravity=g)
    runs = plain_and_one_launch(case, prec, (1, 120, 7))
    assert_same(runs)
    done, _, _, (body,) = runs[0][-1]
    print(name, done, body["status"], flush=True)
    assert 1 < done < 121 and ib_lbm.STATUS[body["status"]] == status


# A light body under the explicit Euler update, which the first step's force
# throws further than 2^31 nodes: the second step finds it outside, whichever
# way it went, and reads nothing there.  (The int of a node so far out saturates.)
# One arc and several, and the pass without arcs
@pytest.mark.parametrize("prec", [ib.FP64, ib.FP32_SHIFTED])
@pytest.mark.parametrize("u", [(0.01, 0.0), (-0.01, 0.0), (0.0, 0.01), (0.01, 0.01), (-0.01, -0.01)])
@pytest.mark.parametrize("arcs", [True, False])
@pytest.mark.parametrize("scheme,kernel,D", [(ib.DF, ib.PESKIN4, 14.0), (ib.DF, ib.HAT, 60.0), (ib.DFC, ib.HAT, 14.0),
                                             (ib.DFC, ib.PESKIN4, 60.0), (ib.MDF, ib.PESKIN4, 60.0)])
def test_a_body_thrown_beyond_every_node_number_is_out_of_range(scheme, kernel, D, arcs, u, prec):
    print(f"thrown {scheme} {kernel} D={D} arcs={arcs} u={u} prec={prec}", flush=True)
    body = dict(xc=50.3, yc=44.6, diameter=D, scheme=scheme, kernel=kernel, mdf_iters=2, motion=ib.FREE,
                density_ratio=1e-13, internal_mass=ib.IM_NONE, integrator=ib.EULER_A1)
    case = box(100, 90, [body], PER)
    pops = ib_cases.random_populations(100, 90, 5, amp=0.0, u=u)
    o = oracle.OracleSim(case)
    o.add_body(body)
    o.set_populations(pops)
    assert o.step(1) == 0 and o.step(1) != 0
    ref = o.body_state()
    o.close()
    assert max(abs(ref["xc"]), abs(ref["yc"])) > 2.0 ** 31
    left = []
    for over in (False, True):
        sim = ib.Sim(case, precision=prec)
        sim.set_overlap(over)
        if not arcs:
            sim.set_spread(ib.SPREAD_ATOMIC)
        sim.set_populations(pops)
        sim.step(1)
        first = sim.populations()
        sim.step(3)
        if arcs:
            assert sim.step_form() == (ib.STEP_ONE if over else ib.STEP_PLAIN)
        st = sim.forces(0, check=False)
        left.append((sim.steps_done, sim.populations(), st))
        sim.close()
        assert left[-1][0] == 1 and ib_lbm.STATUS[st["status"]] == "E_RANGE"
        assert np.array_equal(left[-1][1], first) and np.isfinite(first).all()
        # the force of the first step, times 1 / mass: the schemes' tolerance against the oracle
        d, r = np.array([st["xc"] - 50.3, st["yc"] - 44.6]), np.array([ref["xc"] - 50.3, ref["yc"] - 44.6])
        assert np.abs(d - r).max() <= (1e-9 if prec == ib.FP64 else 1e-3) * np.abs(r).max()
    assert np.array_equal(left[0][1], left[1][1]) and left[0][2] == left[1][2]


@pytest.mark.parametrize("kernel", [ib.HAT, ib.PESKIN4])
def test_a_body_placed_beyond_every_node_number_is_refused(kernel):
    base = dict(xc=50.3, yc=44.6, diameter=14.0, scheme=ib.DF, kernel=kernel, n_markers=40)
    bad = [dict(base, xc=x) for x in (3e9, -3e9, 1e300, float("inf"), float("nan"))]
    bad += [dict(base, yc=y) for y in (3e9, -3e9)] + [dict(base, diameter=1e12)]
    bad += [dict(base, motion=ib.PRESCRIBED_SIN, amp=a, freq=1e-3) for a in ((1e12, 0.0), (0.0, -1e12))]
    sim = ib.Sim(box(100, 90, [], PER))
    for b in bad:
        print(f"refused {b}", flush=True)
        with pytest.raises(ib.IbLbmError) as e:
            sim.add_body(b)
        assert e.value.status == -5
    assert sim.add_body(base) == 0
    sim.close()


# a small disk in a corner of two Zou-He walls: its support holds the node
# diagonally inside the corner, which closes the corner, but not the corner
@pytest.mark.parametrize("prec", [ib.FP64, ib.FP32_SHIFTED])
@pytest.mark.parametrize("kernel", [ib.HAT, ib.PESKIN4])
@pytest.mark.parametrize("east", [False, True])
@pytest.mark.parametrize("north", [False, True])
def test_a_corner_is_closed_before_its_inner_node_is_corrected(north, east, kernel, prec):
    print(f"corner north={north} east={east} kernel={kernel} prec={prec}", flush=True)
    nx, ny, R = 44, 40, 4.0
    low, high = (1.05, 2.05) if kernel == ib.PESKIN4 else (0.05, 1.05)
    x = nx - high - R if east else low + R
    y = ny - high - R if north else low + R
    body = dict(xc=x, yc=y, diameter=2 * R, scheme=ib.DFC, kernel=kernel)
    assert_same(plain_and_one_launch(box(nx, ny, [body], ZOU, ib.TRT), prec, (1, 2, 13, 24)))


# a body in arcs beside one that is too small for them: their passes are two
# launches, and the last to finish completes the case
@pytest.mark.parametrize("scheme", [ib.DF, ib.MDF, ib.DFC])
def test_a_body_in_arcs_beside_one_that_is_not(scheme):
    print(f"mixed bodies scheme={scheme}", flush=True)
    bodies = [dict(xc=x, yc=y, diameter=D, scheme=scheme, kernel=ib.PESKIN4, mdf_iters=3, motion=ib.FREE,
                   density_ratio=1.6, internal_mass=ib.IM_FENG)
              for x, y, D in ((30.3, 40.2, 26.0), (70.4, 38.1, 5.0), (96.2, 60.7, 20.0))]
    case = box(130, 90, bodies, ZOU if scheme == ib.DFC else PER, gravity=(2e-5, 1e-5))
    batch = ib.Batch(ib.FP64)
    sims = [ib.Sim(case), ib.Sim(case)] if scheme != ib.DFC else [ib.Sim(case)]
    ref = oracle.OracleSim(case)
    for b in bodies:
        ref.add_body(b)
    if len(sims) > 1:
        batch.attach(sims[1])
        batch.step(12)
        assert batch.step_form() == ib.STEP_PLAIN
    sims[0].step(12)
    ref.step(12)
    for sim in sims:
        for k in range(3):
            a, b = sim.forces(k), ref.body_state(k)
            assert abs(a["yc"] - b["yc"]) < 1e-12 * b["yc"] and abs(a["vx"] - b["vx"]) < 1e-10 * abs(b["vx"])
        assert rel(sim.populations(), ref.populations()) < F64_FIELD
    assert sims[0].step_form() == ib.STEP_PLAIN
    batch.close()
    for sim in sims:
        sim.close()
    ref.close()


def test_one_launch_steps_after_atomic_spreading():
    """A sim that changes to the atomic scatter and back: the hold rectangles
    of the steps in between are not kept, so the first step after is plain."""
    case = CASES["fast-MDF"]
    print("one-launch after atomic spreading", flush=True)
    out = []
    for over in (False, True):
        sim = ib.Sim(case)
        sim.set_overlap(over)
        sim.step(9)
        sim.set_spread(ib.SPREAD_ATOMIC)
        sim.step(1)
        sim.set_spread(ib.SPREAD_GATHER)
        sim.step(12)
        out.append(sim.populations())
        sim.close()
    assert rel(out[1], out[0]) < F64_FIELD


@pytest.mark.parametrize("prec", [ib.FP64, ib.FP32_SHIFTED])
@pytest.mark.parametrize("graph", [0, 3])
def test_batch_steps_are_bitwise_the_steps_alone(graph, prec):
    """Cases that move, halt, have no body or wait at a target that is raised
    later, stepped by shared launches in calls of odd and even lengths."""
    import torch
    names = ["seam-DF", "open-MDF", "meet-DF", "driven-DFC", "empty-open", "fast-MDF", "arcs-DFC",
             "pair-arcs-DFC", "driven-arcs-DF", "driven-arcs-MDF"]
    targets = [9, 40, 40, 23, 17, 31, 36, 40, 21, 29]
    print(f"batch of one-launch steps graph={graph} prec={prec}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    batch = ib.Batch(prec, stream=stream)
    sims = [ib.Sim(CASES[n], precision=prec, stream=stream) for n in names]
    for s, t in zip(sims, targets):
        batch.attach(s, target=t)
    batch.set_graph(graph)
    for k in (1, 7, 4, 30):
        batch.step(k)
    batch.set_target(sims[0], 14)
    batch.step(5)
    batch.sync()
    assert batch.step_form() == ib.STEP_ONE
    targets[0] = 14
    for n, s, t in zip(names, sims, targets):
        ref = ib.Sim(CASES[n], precision=prec)
        ref.step(t)
        assert ref.step_form() == ib.STEP_ONE
        assert s.steps_done == ref.steps_done, n
        assert np.array_equal(s.populations(), ref.populations()), n
        ref.close()


@pytest.mark.parametrize("graph", [0, 8])
def test_a_batch_changes_behind_queued_steps(graph):
    """Members that join, and a change of the spreading variant, while earlier
    steps are still queued on a stream that the uploads do not wait for."""
    import torch
    print(f"batch changes behind queued steps graph={graph}", flush=True)
    names = ["fast-MDF", "seam-DF", "empty-open", "driven-DFC"]
    stream = torch.cuda.Stream().cuda_stream
    batch = ib.Batch(ib.FP64, stream=stream)
    sims = [ib.Sim(CASES[n], precision=ib.FP64, stream=stream) for n in names]
    batch.set_graph(graph)
    done = [0] * len(sims)
    for i, s in enumerate(sims):
        batch.attach(s)
        batch.step(97)
        for j in range(i + 1):
            done[j] += 97
    batch.set_spread(ib.SPREAD_ATOMIC)
    batch.step(3)
    batch.set_spread(ib.SPREAD_GATHER)
    batch.step(41)
    batch.sync()
    for n, s, k in zip(names, sims, done):
        ref = ib.Sim(CASES[n], precision=ib.FP64)
        ref.step(k)
        ref.set_spread(ib.SPREAD_ATOMIC)
        ref.step(3)
        ref.set_spread(ib.SPREAD_GATHER)
        ref.step(41)
        assert s.steps_done == ref.steps_done == k + 44, n
        # (the order of the atomic sums is open)
        assert rel(s.populations(), ref.populations()) < F64_FIELD, n
        ref.close()
    batch.close()
    for s in sims:
        s.close()


def test_a_sim_changes_behind_queued_steps():
    import torch
    print("sim changes behind queued steps", flush=True)
    out = []
    for queued in (False, True):
        sim = ib.Sim(CASES["fast-MDF"], stream=torch.cuda.Stream().cuda_stream)
        for shape, spread in ((64, 0), (256, 1), (128, 0), (512, 1), (64, 0)):
            sim.step(60)
            if not queued:
                sim.sync()
            sim.set_launch(block_x=shape, block_y=1)
            sim.set_spread(spread)
            sim.step(5)
        out.append(sim.populations())
        sim.close()
    assert rel(out[1], out[0]) < F64_FIELD


def disks(n, D, scheme, **kw):
    """n fixed disks in two rows."""
    p = int(D) + 24
    return box((n + 1) // 2 * p + 40, 2 * p + 10,
               [dict(xc=p * (i // 2 + 0.5) + 20.3, yc=p * (i % 2 + 0.5) + 5.2, diameter=D, scheme=scheme,
                     kernel=ib.PESKIN4, **kw) for i in range(n)], FAR, u_bc=0.04)


# 54 markers of its own an arc (DF, Peskin kernel): 7 or 8 arcs a disk, 56 or 64
# in the launch, on both sides of the number that a sim has in one
@pytest.mark.parametrize("D,form", [(110.0, ib.STEP_ONE), (130.0, ib.STEP_PLAIN)])
def test_sims_on_both_sides_of_the_arcs_in_one_launch(D, form):
    print(f"eight disks of D={D}", flush=True)
    case = disks(8, D, ib.DF)
    out = []
    for over in (False, True):
        sim = ib.Sim(case, precision=ib.FP32_SHIFTED)
        sim.set_overlap(over)
        sim.step(6)
        assert sim.step_form() == (form if over else ib.STEP_PLAIN)
        out.append((sim.populations(), [sim.forces(b) for b in range(8)]))
        sim.close()
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]


# 8 arcs a member: 192 or 200, on both sides of the arcs that may wait at once
@pytest.mark.parametrize("n,form", [(24, ib.STEP_ONE), (25, ib.STEP_PLAIN)])
def test_batches_on_both_sides_of_the_arcs_that_may_wait(n, form):
    print(f"batch of {n} disks", flush=True)
    case = disks(1, 130.0, ib.DF)
    batch = ib.Batch(ib.FP32_SHIFTED)
    sims = [ib.Sim(case, precision=ib.FP32_SHIFTED) for _ in range(n)]
    for s in sims:
        batch.attach(s)
    batch.step(6)
    batch.sync()
    assert batch.step_form() == form
    alone = ib.Sim(case, precision=ib.FP32_SHIFTED)
    alone.step(6)
    for s in sims:
        assert np.array_equal(s.populations(), alone.populations())
    batch.close()


def test_sims_on_several_streams_share_the_arcs_that_may_wait():
    """Three sims of 56 arcs on streams of their own leave 24 of 192: the fourth
    steps in several launches, until another gives its arcs back; one on the
    stream of another needs none of its own."""
    import torch
    print("arcs shared by streams", flush=True)
    case = disks(8, 110.0, ib.DF)
    streams = [torch.cuda.Stream().cuda_stream for _ in range(4)]
    sims = [ib.Sim(case, precision=ib.FP32_SHIFTED, stream=st) for st in streams + streams[:1]]
    for s in sims:
        s.step(6)
    assert [s.step_form() for s in sims] == [ib.STEP_ONE] * 3 + [ib.STEP_PLAIN, ib.STEP_ONE]
    sims[1].close()
    for s in (sims[0], sims[2], sims[3], sims[4]):
        s.set_launch()  # plans its steps anew
        s.step(5)
        assert s.step_form() == ib.STEP_ONE
    pops = [s.populations() for s in (sims[0], sims[2], sims[3], sims[4])]
    assert all(np.array_equal(p, pops[0]) for p in pops)
    for s in sims:
        s.close()


def test_sims_on_four_streams_at_the_arcs_that_may_wait():
    """160 arcs on as many streams as have a hardware queue, in workgroups of 256
    and 512 threads."""
    import torch
    print("four streams", flush=True)
    cases = [disks(8, 110.0, ib.DF), disks(8, 36.0, ib.MDF, mdf_iters=5),
             disks(8, 110.0, ib.DF), disks(8, 60.0, ib.DFC)]
    sims = [ib.Sim(c, precision=ib.FP32_SHIFTED, stream=torch.cuda.Stream().cuda_stream) for c in cases]
    for _ in range(20):
        for s in sims:
            s.step(25)
    for s, c in zip(sims, cases):
        assert s.step_form() == ib.STEP_ONE
        alone = ib.Sim(c, precision=ib.FP32_SHIFTED)
        alone.step(500)
        assert [s.forces(b) for b in range(8)] == [alone.forces(b) for b in range(8)]
        assert np.array_equal(s.populations(), alone.populations())
        alone.close()


def test_the_tuner_times_nothing_that_one_launch_steps_ignore(monkeypatch):
    from paper_2609_02298_amd import autotune
    print("tuner and one-launch steps", flush=True)
    shape = dict(block_x=64, block_y=2, rows_per_thread=1, xcd_remap=1)
    monkeypatch.setattr(autotune, "_cache", {"other": {}})
    monkeypatch.setattr(autotune, "tune", lambda *a, **k: dict(shape))
    timed = []
    monkeypatch.setattr(autotune, "time_step", lambda c, p, sh, n: timed.append("step") or 1.0)
    monkeypatch.setattr(autotune, "time_ib", lambda c, p, t, n, sh: timed.append("ib") or 1.0)
    case = disks(1, 20.0, ib.MDF, mdf_iters=5)
    assert autotune.tune_step(case, ib.FP64) == dict(shape, ib_threads=0)
    assert not timed and set(autotune._cache) == {"other"}
    # a coupled body keeps the launches that the shape is for
    autotune.tune_step(disks(1, 20.0, ib.MDF, mdf_iters=5, mdf_coupled=1), ib.FP64)
    assert set(timed) == {"step", "ib"} and len(autotune._cache) == 3


# Peskin stencils are loaded by columns, the hat's by rows: a body on a seam of the
# lattice's storage (64 columns), at each offset of a stencil from it
@pytest.mark.parametrize("scheme", [ib.DF, ib.MDF, ib.DFC])
@pytest.mark.parametrize("xc", [63.1, 64.2, 65.3, 66.4])
@pytest.mark.parametrize("kernel", [ib.PESKIN4, ib.HAT])
def test_columns_across_a_storage_seam_match_the_oracle(kernel, scheme, xc):
    print(f"seam scheme={scheme} kernel={kernel} xc={xc}", flush=True)
    case = box(140, 60, [dict(xc=xc, yc=30.3, diameter=9.0, scheme=scheme, kernel=kernel, mdf_iters=5)],
               FAR, u_bc=0.05)
    sim, ref = ib.Sim(case), oracle.OracleSim(case)
    ref.add_body(case["bodies"][0])
    sim.step(9)
    ref.step(9)
    a, b = sim.forces(0), ref.body_state(0)
    assert abs(a["fx"] - b["fx"]) < F64_DRAG * abs(b["fx"])
    assert rel(sim.populations(), ref.populations()) < F64_FIELD
    sim.close()
    ref.close()


# a batch's steps take one launch up to 20 M nodes (FP32) or 40 M (FP64), several
# beyond: on both sides of the line the members are bitwise the sims alone
@pytest.mark.parametrize("prec,ny", [(ib.FP32_SHIFTED, 2220), (ib.FP32_SHIFTED, 2225),
                                     (ib.FP64, 4440), (ib.FP64, 4450)])
def test_batch_steps_on_both_sides_of_the_size_line(prec, ny):
    print(f"batch of 2 x 4500 x {ny}, precision {prec}", flush=True)
    bodies = [dict(xc=900.3, yc=ny / 2 + 0.4, diameter=60.0, scheme=ib.DFC, kernel=ib.HAT)]
    members = [box(4500, ny, bodies, FAR, ib.CMMRT, u_bc=0.05), box(4500, ny, [], FAR, ib.BGK, u_bc=0.05)]
    batch = ib.Batch(prec)
    sims = [ib.Sim(m, precision=prec) for m in members]
    for s in sims:
        batch.attach(s)
    batch.step(5)
    batch.sync()
    assert batch.step_form() == (ib.STEP_ONE if ny in (2220, 4440) else ib.STEP_PLAIN)
    for s, m in zip(sims, members):
        alone = ib.Sim(m, precision=prec)
        alone.step(5)
        assert all(np.array_equal(a, b) for a, b in zip(s.fields(), alone.fields()))
        if m["bodies"]:
            assert s.forces(0)["fx"] == alone.forces(0)["fx"]
        alone.close()
    batch.close()
    for s in sims:
        s.close()
