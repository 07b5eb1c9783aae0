"""Runs of two or more steps, which take two steps a launch (binary64 and
binary32 storage without a source), against steps taken one by one (bit for
bit: a cell's arithmetic and its order are the same in both) and against the
oracle (binary64, max-norm relative to max |f~| <= 1e-12, the bound of the
one-step parity tests).

Sizes at the edges of the 60-column strips and of row chunks, meshes of one to
three cells (wrapped more than once, ghosts of ghosts), every pair of wall
kinds.  A Dirichlet axis beside a periodic one steps one at a time; it is run
here too."""
import numpy as np
import pytest

import paper_1906_11036_amd as dg
from oracle import Oracle
from paper_1906_11036_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 1), (1, 3), (3, 2), (59, 5), (60, 7), (61, 4), (62, 9), (63, 3), (120, 2), (121, 33), (181, 6)]
WALLS = [(W.PERIODIC, W.PERIODIC), (W.DIRICHLET, W.DIRICHLET), (W.MIRROR, W.MIRROR), (W.PERIODIC, W.MIRROR),
         (W.MIRROR, W.PERIODIC), (W.DIRICHLET, W.MIRROR), (W.MIRROR, W.DIRICHLET), (W.PERIODIC, W.DIRICHLET)]


def solver(p, storage, rows, wpb, rings):
    s = dg.Solver(p, storage=storage)
    s.set_launch(rows, wpb, 0, 1)
    if rings is not None:
        s.set_dirichlet(rings)
    s.set_phi(p.phi0)
    return s


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("q", [9, 5])
def test_two_steps_a_launch(nx, ny, q):
    n = 7   # a graph of four (two launches), a pair and a single step
    for i, (bcx, bcy) in enumerate(WALLS):
        p = W.random_problem(900 + i + 10 * q, nx, ny, q=q, bcx=bcx, bcy=bcy, stretched=i % 2 == 1, bdeg=1 + i % 3,
                             ddeg=1)
        if W.MIRROR in (bcx, bcy):   # a wall moves no mass: no convection through it
            p.bx, p.by = (0.0, 0.1), (0.0, 0.1)
        rings = p.rings(n)
        print(f"case {nx}x{ny} q={q} bc=({bcx},{bcy})", flush=True)
        o = Oracle(p)
        o.step(n, rings)
        ref = o.get_f()
        for storage in ("f64", "f32"):
            one = solver(p, storage, 4, 1, rings)
            for _ in range(n):
                one.step(1)
            want = one.get_f()
            if storage == "f64":
                assert np.abs(want - ref).max() <= 1e-12 * np.abs(ref).max()
            for rows, wpb in ((1, 1), (2, 4), (5, 2), (64, 1)):
                two = solver(p, storage, rows, wpb, rings)
                two.step(n)
                assert np.array_equal(two.get_f(), want), (storage, rows)
                assert two.diag()["step"] == n


def test_state_after_an_odd_number_of_launches():
    """Read-outs, checkpoints and further runs find the state in either buffer:
    2, 6 (a graph from the other buffer), 1 and 4 steps in turn."""
    p = W.random_problem(77, 130, 41, bdeg=2, ddeg=2)
    for storage in ("f64", "f32"):
        a, e = (solver(p, storage, 3, 1, None) for _ in range(2))
        for n in (2, 6, 1, 4, 3):
            a.step(n)
            for _ in range(n):
                e.step(1)
            assert np.array_equal(a.get_f(), e.get_f())
            assert np.array_equal(a.get_phi(), e.get_phi())
            assert a.diag()["mass"] == e.diag()["mass"]
            b = solver(p, storage, 2, 1, None)
            b.restore(a.checkpoint())
            b.step(5)
            c = solver(p, storage, 2, 1, None)
            c.restore(e.checkpoint())
            for _ in range(5):
                c.step(1)
            assert np.array_equal(b.get_f(), c.get_f())


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.MIRROR])
def test_captured_steps_can_be_replayed(storage, bc):
    """An even number of steps captured by the caller ends in the buffer it began
    in, so each replay advances the state (eager work and reads between the
    replays)."""
    import torch
    p = W.random_problem(78, 130, 41, bcx=bc, bcy=bc, bdeg=1, ddeg=1)
    if bc == W.MIRROR:
        p.bx, p.by = (0.0, 0.1), (0.0, 0.1)
    print(f"case captured steps {storage} bc={bc}", flush=True)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        for n in (2, 4, 6):
            a, e = (solver(p, storage, 3, 1, None) for _ in range(2))
            for s in (a, e):
                s.step(2)
            st.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st):
                a.step(n)
            for _ in range(4):
                g.replay()
                e.step(n)
                st.synchronize()
                assert np.array_equal(a.get_f(), e.get_f()), n


@pytest.mark.parametrize("storage", ["f64", "f32", "f16neq"])
def test_runs_from_every_phase_and_either_buffer(storage):
    """Runs that start at any step, with the state in either buffer (two steps a
    launch, or a state restored at an odd step): one captured graph serves both."""
    p = W.random_problem(79, 130, 41, bdeg=2, ddeg=2)
    print(f"case runs from every phase {storage}", flush=True)
    a, e = (solver(p, storage, 3, 1, None) for _ in range(2))
    for n in (1, 6, 2, 11, 5, 40, 3, 9):
        a.step(n)
        for _ in range(n):
            e.step(1)
        assert np.array_equal(a.get_f(), e.get_f()), n
    a.step(1)
    blob = a.checkpoint()
    b, c = (solver(p, storage, 2, 1, None) for _ in range(2))
    for s in (b, c):
        s.restore(blob)
    b.step(41)
    for _ in range(41):
        c.step(1)
    assert b.info()["graph_steps"] >= 36
    assert np.array_equal(b.get_f(), c.get_f())
