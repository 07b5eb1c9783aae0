"""GPU parity of the one-dimensional D1Q3 path (B = b(x, t) phi, D = d(t) phi,
C = 0, R from dB/dt; Remark 3, Example 4.6) against the 1-D CPU oracle,
through the C ABI of include/dugks1d.h."""
import math

import numpy as np
import pytest

import paper_1906_11036_amd as dg
from oracle import Oracle1D
from paper_1906_11036_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS32 = float(np.finfo(np.float32).eps)
P, D = W.PERIODIC, W.DIRICHLET1


def say(*a):
    print(*a, flush=True)


def rel_max(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


@pytest.mark.parametrize("n", [1, 5, 61, 62, 63, 64, 123, 124, 125, 300])
@pytest.mark.parametrize("bc", [P, D])
@pytest.mark.parametrize("stretched", [False, True])
def test_fp64_matches_oracle(n, bc, stretched):
    """Uniform meshes take the kernel's table-free instantiation, stretched ones
    the per-cell geometry tables."""
    p = W.random_problem1d(900 + n, n, bc=bc, stretched=stretched)
    say(f"case 1d f64 n={n} bc={bc} stretched={stretched}")
    s = dg.Solver1D(p, "f64")
    s.set_phi(p.phi0)
    s.step(7)
    o = Oracle1D(p)
    o.step(7)
    assert rel_max(s.get_f(), o.get_f()) <= 1e-12
    assert rel_max(s.get_phi_prev(), o.get_phi_prev()) <= 1e-12
    r = s.reduce()
    assert abs(r["mass"] - o.mass()) <= 1e-12 * abs(o.mass())


@pytest.mark.parametrize("bc", [P, D])
def test_set_state_one_step(bc):
    n = 200
    p = W.random_problem1d(77, n, bc=bc, stretched=True)
    rng = np.random.default_rng(3)
    f = np.stack([0.6 + 0.05 * rng.standard_normal(n), 0.2 + 0.05 * rng.standard_normal(n),
                  0.2 + 0.05 * rng.standard_normal(n)])
    pp = f.sum(axis=0) + 0.01 * rng.standard_normal(n)
    s = dg.Solver1D(p, "f64")
    s.set_state(f, pp)
    s.step(1)
    o = Oracle1D(p)
    o.set_state(f, pp)
    o.step(1)
    assert rel_max(s.get_f(), o.get_f()) <= 1e-12


def test_dirichlet_data_in_pieces_and_exhaustion():
    """Ghost data given in three pieces equals one table (the pair of the last
    step of a piece carries over as the ghosts' previous values)."""
    p = W.random_problem1d(31, 90, bc=D)
    s = dg.Solver1D(p, "f64")
    s.set_phi(p.phi0)
    table = s.ghost_table(9)
    s.set_dirichlet(table[:3])
    s.step(3, auto_ghosts=False)
    s.set_dirichlet(table[3:5])
    with pytest.raises(dg.DugksError):
        s.step(3, auto_ghosts=False)          # only 2 pairs left: nothing is stepped
    s.step(2, auto_ghosts=False)
    s.set_dirichlet(table[5:9])
    s.step(4, auto_ghosts=False)
    o = Oracle1D(p)
    o.step(9)
    assert rel_max(s.get_f(), o.get_f()) <= 1e-12
    assert s.info()["steps"] == 9


def test_fokker_planck_gre_equals_oracle():
    """Example 4.6 (closed form eq. 4.6.3 from t = 0.5 to 1, Dirichlet data from
    it), dx = 1/20, dt = 1e-5 as in the paper's convergence protocol."""
    n, dt = 200, 1e-5
    p = W.fokker_planck_problem(n, t0=0.5, c=0.5 * (10.0 / n) / dt, cfl=0.5)
    s = dg.Solver1D(p, "f64")
    s.set_phi(p.phi0)
    o = Oracle1D(p)
    nst = int(round(0.5 / o.dt))
    s.step(nst)
    o.step(nst)
    exact = W.fokker_planck_exact(p.centres(), o.time)
    gre = s.reduce(exact)["gre"]
    gre_o = o.errors(exact)[0]
    dphi = rel_max(s.get_phi(), o.get_phi())
    say(f"  Fokker-Planck n={n}: GRE gpu {gre:.6e} oracle {gre_o:.6e}, max rel phi diff {dphi:.1e} "
        f"after {nst} steps")
    # 5e4 steps, each with rounding differences of a few ulp (FMA contraction, the
    # closed-form transforms against the oracle's literal route, whose f from f~
    # divides by 1 + dt/(2 lambda) ~ 11 here): phi agrees to 1e-10 of max |phi|,
    # so the GRE (3.6e-4 of |phi|) agrees to 1e-10 / 3.6e-4 < 1e-6 relative
    assert dphi <= 1e-10
    assert abs(gre - gre_o) <= 1e-6 * gre_o
    assert gre <= 4e-4


@pytest.mark.parametrize("bc", [P, D])
@pytest.mark.parametrize("stretched", [False, True])
def test_fp32_against_oracle(bc, stretched):
    p = W.random_problem1d(55, 400, bc=bc, stretched=stretched)
    steps = 60
    s = dg.Solver1D(p, "f32")
    s.set_phi(p.phi0)
    s.step(steps)
    o = Oracle1D(p)
    o.step(steps)
    ref = o.get_phi()
    err = float(np.sqrt(((s.get_phi() - ref) ** 2).sum() / (ref ** 2).sum()))
    say(f"  1d f32 bc={bc}: rel-L2 {err:.2e} (bound {2 * steps * EPS32:.2e})")
    assert err <= 2 * steps * EPS32


@pytest.mark.parametrize("storage,tol", [("f32", 2e-6), ("f64", 1e-12)])
def test_full_size_one_step_sampled_1d(storage, tol):
    """The benchmark instance (2^26 cells, Example 4.6 on [-2, 8]) in its launch:
    one step from a seeded non-equilibrium state, checked at sampled cells
    (walls, wave seams, random cells) against the oracle."""
    p = W.workload1d("fokker_planck_64m")
    n = p.nx
    say(f"case full size 1-D n={n} {storage}")
    rng = np.random.default_rng(2026)
    phi = p.phi0
    f = np.stack([phi * (2 / 3), phi / 6, phi / 6]) + 1e-3 * rng.standard_normal((3, n))
    pp = phi + 1e-4 * rng.standard_normal(n)
    s = dg.Solver1D(p, storage)
    s.set_state(f, pp)
    f_used = s.get_f()              # the stored state (rounded to the storage format)
    pp_used = s.get_phi_prev()
    s.step(1)
    gpu = s.get_f()
    s.close()
    o = Oracle1D(p)
    o.set_state(f_used, pp_used)
    cells = set([0, 1, 2, 60, 61, 62, 63, 123, 124, n - 3, n - 2, n - 1, n // 2])
    cells |= set(int(v) for v in rng.integers(0, n, 600))
    cells = np.array(sorted(cells))
    ref = o.step_cells(cells)
    err = float(np.abs(gpu[:, cells].T - ref).max() / np.abs(ref).max())
    say(f"  sampled max rel err {err:.2e} over {len(cells)} cells")
    assert err <= tol


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 55, 56, 57, 59, 60, 61, 64, 112, 113, 900])
@pytest.mark.parametrize("bc", [P, D])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_four_steps_a_launch(n, bc, storage):
    """Runs of four or more steps take four a launch (56 cells a wave): bit for bit
    the steps taken one by one on uniform meshes (meshes of fewer cells than a
    wave's halo and the edges of its strips among them)."""
    p = W.random_problem1d(950 + n, n, bc=bc)
    say(f"case 1d four steps n={n} bc={bc} {storage}")
    a, e = dg.Solver1D(p, storage), dg.Solver1D(p, storage)
    for s in (a, e):
        s.set_phi(p.phi0)
    for steps in (9, 4, 6):
        if bc == D:
            g = a.ghost_table(steps)
            for s in (a, e):
                s.set_dirichlet(g)
        a.step(steps, auto_ghosts=False)
        for _ in range(steps):
            e.step(1, auto_ghosts=False)
        assert np.array_equal(a.get_f(), e.get_f())
        assert np.array_equal(a.get_phi_prev(), e.get_phi_prev())


@pytest.mark.parametrize("n", [1, 2, 3, 5, 55, 56, 57, 64, 113, 400, 900])
@pytest.mark.parametrize("bc", [P, D])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_four_steps_a_launch_on_stretched_meshes(n, bc, storage):
    """The same on stretched meshes, whose geometry comes from tables: past a
    periodic seam a lane steps the cell that it wraps to with the factors of
    that cell's own faces."""
    p = W.random_problem1d(970 + n, n, bc=bc, stretched=True)
    say(f"case 1d four steps, stretched, n={n} bc={bc} {storage}")
    a, e = dg.Solver1D(p, storage), dg.Solver1D(p, storage)
    for s in (a, e):
        s.set_phi(p.phi0)
    for steps in (8, 9, 40):
        if bc == D:
            g = a.ghost_table(steps)
            for s in (a, e):
                s.set_dirichlet(g)
        a.step(steps, auto_ghosts=False)
        for _ in range(steps):
            e.step(1, auto_ghosts=False)
        assert np.array_equal(a.get_f(), e.get_f())
        assert np.array_equal(a.get_phi_prev(), e.get_phi_prev())


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_captured_steps_can_be_replayed(storage):
    """An even number of steps captured by the caller ends in the buffer it began
    in, so each replay advances the state (b and d constant in time)."""
    import torch
    p = W.random_problem1d(960, 200, bc=P)
    p.coef = (0.0, 0.0, 0.3, 0.0, 0.0, 0.8, 0.0)
    say(f"case 1d captured steps {storage}")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        for n in (2, 4, 6):
            a, e = dg.Solver1D(p, storage), dg.Solver1D(p, storage)
            for s in (a, e):
                s.set_phi(p.phi0)
                s.step(4)
            st.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st):
                a.step(n)
            for _ in range(4):
                g.replay()
                e.step(n)
                st.synchronize()
                assert np.array_equal(a.get_f(), e.get_f()), n


def test_large_host_read_out():
    """Host read-outs of many megabytes go through pinned chunks emptied by several
    threads: every value arrives, at sizes that are no multiple of a chunk or of
    the threads (and twice from one solver)."""
    for n in ((1 << 21) + 5, (1 << 22) - 3):
        p = W.random_problem1d(41, n, bc=P)
        rng = np.random.default_rng(n)
        f, prev = rng.standard_normal((3, n)), rng.standard_normal(n)
        s = dg.Solver1D(p, "f64")
        for _ in range(2):
            s.set_state(f, prev)
            assert np.array_equal(s.get_f(), f)
            assert np.array_equal(s.get_phi_prev(), prev)
            f, prev = f[:, ::-1].copy(), prev[::-1].copy()
