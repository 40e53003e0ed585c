"""GPU parity of the batched path (many independent 1D Euler problems of
uneven size, tenom_batch_*) against the oracle run problem by problem, and
its invariants: every tile shape, the graph replay, the persistent launch
and per-problem launches give the same bits; the autotuner leaves the state
alone; an empty batch is a no-op."""
import numpy as np
import pytest

import workloads as W
from oracle import exact_riemann as ER
from parity import (RTOL, assert_close_fields, band_faces, conditioning_tol, faces_to_cells, field_scale,
                    require_gpu, to_dev, to_host, ulp_perturbed)

pytestmark = pytest.mark.gpu

GAMMA = 1.4
CFL = 0.4
# ragged sizes around the tile boundaries (63/64/65, 127/128/129, 255/256/257,
# 511/512/513) and the smallest admissible problems
SIZES = [8, 9, 13, 63, 64, 65, 127, 128, 129, 254, 255, 256, 257, 300, 511, 512, 513, 700, 1023, 1025]


def ragged_batch(sizes, seed0=0):
    """One seeded Riemann problem per entry (states as W.riemann_states),
    packed end to end; dx = 1/n on [0, 1]."""
    parts, dx, states = [], [], []
    for p, n in enumerate(sizes):
        left, right = W.riemann_states(seed0 + p)
        U, h = W.riemann_problem(int(n), left, right, gamma=GAMMA)
        parts.append(U)
        dx.append(h)
        states.append((left, right))
    return np.concatenate(parts, axis=1), np.array(dx), states


def problem(U, plan, p):
    a, b = plan.offsets[p], plan.offsets[p + 1]
    return np.ascontiguousarray(U[:, a:b])


def grid_of(n, dx, bc):
    return dict(ndim=1, n=[int(n)], dx=[float(dx)], bc=[bc], system=1)


def rk3_excluded(orc, U, grid, scheme, lim, C_T, dt):
    """Cells whose step depends on a face in the cutoff band at any stage."""
    L0 = orc.flux_divergence(U, grid, scheme, lim, C_T, GAMMA)
    U1 = U + dt * L0
    L1 = orc.flux_divergence(U1, grid, scheme, lim, C_T, GAMMA)
    U2 = 0.75 * U + 0.25 * (U1 + dt * L1)
    n = grid["n"][0]
    excl = np.zeros(n, dtype=bool)
    for S in (U, U1, U2):
        _, _, bd = orc.reconstruct_faces(S, grid, scheme, lim, C_T, GAMMA, 0)
        excl |= faces_to_cells(band_faces(bd), 0, n, grid["bc"][0] == 0, 3 * (scheme & 0xFF) // 2)
    return excl


@pytest.fixture(scope="module")
def T():
    require_gpu()
    import paper_2010_13289_amd as T
    return T


# name, scheme, limiter, C_T, bc
CASES = [
    ("tvd8_trans", 8, 2, 1e-7, 1),
    ("mp8_trans", 8, 1, 1e-7, 1),
    ("mp6_periodic", 6, 1, 1e-5, 0),
    ("teno8a_va_trans", 8 | 0x100, 4, 0.0, 1),
    ("teno6_classic_periodic", 6, 0, 1e-5, 0),
    ("tvd5_8_periodic", 8, 3, 1e-7, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_batch_steps_match_the_oracle(T, orc, case):
    """Three steps; each compared problem by problem with the oracle's step
    from the same input with the step size the device chose, which must be
    the oracle's CFL step."""
    name, scheme, lim, C_T, bc = case
    U, dx, _ = ragged_batch(SIZES, seed0=11)
    plan = T.BatchPlan(SIZES, dx, bc)
    Ud = to_dev(U)
    for step in range(3):
        print(f"[batch] {name} step {step}", flush=True)
        Uin = to_host(Ud)
        plan.rk3(Ud, scheme, lim, C_T, GAMMA, CFL, steps=1)
        t, dt = plan.times()
        Ug = to_host(Ud)
        for p, n in enumerate(SIZES):
            g = grid_of(n, dx[p], bc)
            Up = problem(Uin, plan, p)
            assert dt[p] == pytest.approx(CFL / orc.max_wave_speed(Up, g, GAMMA), rel=1e-13)
            Uo = orc.rk3_step(Up, g, scheme, lim, C_T, GAMMA, dt[p])
            excl = rk3_excluded(orc, Up, g, scheme, lim, C_T, dt[p])
            assert excl.sum() < n // 2, f"problem {p}: {excl.sum()} band cells"
            assert_close_fields(problem(Ug, plan, p), Uo, exclude=excl, what=f"{name} step {step} problem {p}")
    t, _ = plan.times()
    assert np.all(t > 0)
    plan.close()


# problems of K and K + 1 cells (six points) between larger ones
SMALL = [6, 7, 6, 12, 7, 255, 256, 257]


@pytest.mark.parametrize("bc", [0, 1], ids=["periodic", "transmissive"])
def test_smallest_problems_match_the_oracle(T, orc, bc):
    """Six-point problems as short as the stencil: two steps compared with
    the oracle problem by problem, and the persistent launch of the same two
    steps in the same bits."""
    U, dx, _ = ragged_batch(SMALL, seed0=41)
    plan = T.BatchPlan(SMALL, dx, bc)
    pers = T.BatchPlan(SMALL, dx, bc)
    Ud = to_dev(U)
    for step in range(2):
        print(f"[batch small] bc={bc} step {step}", flush=True)
        Uin = to_host(Ud)
        plan.rk3(Ud, 6, T.LIM_MP, 1e-5, GAMMA, CFL, steps=1)
        _, dt = plan.times()
        Ug = to_host(Ud)
        for p, n in enumerate(SMALL):
            g = grid_of(n, dx[p], bc)
            Up = problem(Uin, plan, p)
            assert dt[p] == pytest.approx(CFL / orc.max_wave_speed(Up, g, GAMMA), rel=1e-13)
            Uo = orc.rk3_step(Up, g, 6, 1, 1e-5, GAMMA, dt[p])
            excl = rk3_excluded(orc, Up, g, 6, 1, 1e-5, dt[p])
            assert excl.sum() < max(n // 2, 1), f"problem {p}: {excl.sum()} band cells"
            assert_close_fields(problem(Ug, plan, p), Uo, exclude=excl, what=f"small bc={bc} step {step} problem {p}")
    B = to_dev(U)
    pers.rk3_persistent(B, 6, T.LIM_MP, 1e-5, GAMMA, CFL, steps=2)
    assert np.array_equal(to_host(B), to_host(Ud)), "persistent launch differs from the eager steps"
    plan.close()
    pers.close()


def test_every_tile_gives_the_same_bits(T):
    U, dx, _ = ragged_batch(SIZES, seed0=3)
    plan = T.BatchPlan(SIZES, dx, 1)
    ref = None
    for tile in range(T.BATCH_TILES):
        print(f"[batch] tile {tile} {T.batch_tile_shape(tile)}", flush=True)
        plan.tile = tile
        Ud = to_dev(U)
        plan.rk3(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=2)
        out = to_host(Ud)
        if ref is None:
            ref = out
        assert np.array_equal(out, ref), f"tile {tile} differs"
    plan.close()


def test_graph_replays_match_eager_steps(T):
    """The captured graph equals the eager enqueue in every bit, on the
    first launch and on replays with other device work in between."""
    import torch
    U, dx, _ = ragged_batch(SIZES, seed0=5)
    plan = T.BatchPlan(SIZES, dx, 1)
    A = to_dev(U)
    B = to_dev(U)
    other = to_dev(U)
    for replay in range(3):
        print(f"[batch] graph replay {replay}", flush=True)
        plan.rk3(A, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=4)
        plan.rk3_graph(B, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=4)
        assert np.array_equal(to_host(A), to_host(B)), f"replay {replay}"
        # unrelated eager work and a synchronisation between replays
        plan.rk3(other, 6, T.LIM_TVD5, 1e-5, GAMMA, CFL, steps=1)
        other.mul_(1.0)
        torch.cuda.synchronize()
    plan.close()


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_persistent_launch_matches_eager_steps(T, case):
    """One persistent launch of 5 steps equals 5 eager steps in every bit,
    with the same clocks and last steps (wrapped periodic problems of at
    most 256 cells, multi-segment problems, both boundary rules)."""
    name, scheme, lim, C_T, bc = case
    U, dx, _ = ragged_batch(SIZES, seed0=21)
    eager = T.BatchPlan(SIZES, dx, bc)
    pers = T.BatchPlan(SIZES, dx, bc)
    A = to_dev(U)
    B = to_dev(U)
    print(f"[batch persistent] {name}", flush=True)
    eager.rk3(A, scheme, lim, C_T, GAMMA, CFL, steps=5)
    pers.rk3_persistent(B, scheme, lim, C_T, GAMMA, CFL, steps=5)
    assert np.array_equal(to_host(A), to_host(B)), f"{name}: state differs"
    ta, da = eager.times()
    tb, db = pers.times()
    assert np.array_equal(ta, tb) and np.array_equal(da, db), f"{name}: clocks differ"
    eager.close()
    pers.close()


def test_persistent_launch_in_a_captured_graph(T):
    """The persistent launch captured in a graph and replayed three times,
    with other device work between the replays, equals the eager launch in
    every bit each time (the plan's queue is clear again after each launch)."""
    import torch
    U, dx, _ = ragged_batch(SIZES, seed0=27)
    plan = T.BatchPlan(SIZES, dx, 1)
    ref_plan = T.BatchPlan(SIZES, dx, 1)
    Us = to_dev(U)
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            plan.rk3_persistent(Us, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=2)
    torch.cuda.current_stream().wait_stream(side)
    R = to_dev(U)
    for replay in range(3):
        print(f"[batch persistent graph] replay {replay}", flush=True)
        Us.copy_(to_dev(U) if replay == 0 else Us)
        g.replay()
        ref_plan.rk3_persistent(R, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=2)
        torch.cuda.synchronize()
        assert torch.equal(Us, R), f"replay {replay} differs"
        R.mul_(1.0)  # unrelated work between replays
        torch.cuda.synchronize()
    plan.close()
    ref_plan.close()


def test_problem_ranges_match_the_whole_batch(T):
    """One launch per problem (first = p, count = 1) gives the same bits and
    clocks as one launch over the batch."""
    sizes = SIZES[:12]
    U, dx, _ = ragged_batch(sizes, seed0=21)
    whole = T.BatchPlan(sizes, dx, 1)
    single = T.BatchPlan(sizes, dx, 1)
    A = to_dev(U)
    B = to_dev(U)
    whole.rk3(A, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=3)
    for p in range(len(sizes)):
        single.rk3(B, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=3, first=p, count=1)
    assert np.array_equal(to_host(A), to_host(B))
    assert np.array_equal(whole.times()[0], single.times()[0])
    # a range touches only its own problems
    C_ = to_dev(U)
    whole.rk3(C_, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=1, first=3, count=2)
    out = to_host(C_)
    a, b = whole.offsets[3], whole.offsets[5]
    assert np.array_equal(out[:, :a], U[:, :a]) and np.array_equal(out[:, b:], U[:, b:])
    assert not np.array_equal(out[:, a:b], U[:, a:b])
    whole.close()
    single.close()


def test_autotune_keeps_state_and_clocks(T):
    U, dx, _ = ragged_batch(SIZES, seed0=8)
    plan = T.BatchPlan(SIZES, dx, 1)
    Ud = to_dev(U)
    plan.rk3(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=1)
    before = to_host(Ud)
    t0, dt0 = plan.times()
    best, ms = plan.autotune(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=2)
    assert 0 <= best < T.BATCH_TILES and plan.tile == best
    assert all(m > 0 for m in ms) and ms[best] == min(ms)
    assert np.array_equal(to_host(Ud), before)
    t1, dt1 = plan.times()
    assert np.array_equal(t0, t1) and np.array_equal(dt0, dt1)
    plan.close()


def test_empty_batch_and_errors(T):
    import torch
    plan = T.BatchPlan([], [], 1)
    assert plan.total == 0
    U = torch.empty((3, 0), dtype=torch.float64, device="cuda")
    plan.rk3(U, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=5)
    plan.rk3_graph(U, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=5)
    plan.rk3_persistent(U, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=5)
    assert plan.autotune(U, 8, T.LIM_MP, 1e-7, GAMMA, CFL)[0] == plan.tile
    assert plan.times()[0].size == 0
    plan.close()
    # a 6-cell problem admits K = 6 but not K = 8
    Ub, dx, _ = ragged_batch([6, 40])
    plan = T.BatchPlan([6, 40], dx, 1)
    Ud = to_dev(Ub)
    plan.rk3(Ud, 6, T.LIM_MP, 1e-5, GAMMA, CFL)
    for args, code in (((8, T.LIM_MP, 1e-7, GAMMA, CFL), T.EINVAL), ((6, T.LIM_MP, 1e-5, GAMMA, 0.0), T.EINVAL),
                       ((6, 99, 1e-5, GAMMA, CFL), T.EUNSUPPORTED), ((6, T.LIM_MP, 1e-5, 1.0, CFL), T.EINVAL)):
        with pytest.raises(T.TenomError) as e:
            plan.rk3(Ud, *args)
        assert e.value.code == code
    with pytest.raises(T.TenomError) as e:
        plan.rk3(Ud, 6, T.LIM_MP, 1e-5, GAMMA, CFL, first=1, count=2)
    assert e.value.code == T.EINVAL
    with pytest.raises(T.TenomError):
        plan.rk3(Ud, 6, T.LIM_MP, 1e-5, GAMMA, CFL, steps=-1)
    torch.cuda.synchronize()
    plan.close()


def test_batched_4096_problems_graph_100_steps(T, orc):
    """The benchmark's batch: 4096 problems, n log-uniform in [256, 16384],
    TENO8-M-MP, 100 steps in one graph launch.  Checks: every problem equals
    the oracle run problem by problem on 12 sampled problems (tolerance
    from the oracle's own sensitivity to one-ulp differences at every step
    of the run; per-step parity is test_batch_steps_match_the_oracle's),
    conservation
    of every problem to round-off (no wave reaches an end in 100 steps),
    positivity, and the exact solution as a loose physics check."""
    import torch
    sizes = W.batched_riemann_sizes()
    U, dx, states = ragged_batch(sizes)
    plan = T.BatchPlan(sizes, dx, 1)
    Ud = to_dev(U)
    best, ms = plan.autotune(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=1)
    print(f"[batch 4096] autotuned tile {best} {T.batch_tile_shape(best)}, ms/step {ms}", flush=True)
    plan.rk3_graph(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=100)
    torch.cuda.synchronize()
    t, _ = plan.times()
    Ug = to_host(Ud)
    # the persistent launch: the same 100 steps in one kernel, the same bits
    pers = T.BatchPlan(sizes, dx, 1)
    Up = to_dev(U)
    print("[batch 4096] persistent launch, 100 steps", flush=True)
    pers.rk3_persistent(Up, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=100)
    assert np.array_equal(to_host(Up), Ug), "persistent launch differs from the graph"
    assert np.array_equal(pers.times()[0], t)
    pers.close()
    del Up
    assert np.all(np.isfinite(Ug)) and np.all(Ug[0] > 0)
    rho, m, E = Ug
    assert np.all(E - 0.5 * m * m / rho > 0)
    # conservation per problem: no wave reaches an end in 100 steps (only
    # round-off-level precursors do), so sum(U) changes by the flux through
    # the two ends, t (F(U_first) - F(U_last)) / dx
    seg_sum = lambda A: np.add.reduceat(A, plan.offsets[:-1], axis=1)
    before, after = seg_sum(U), seg_sum(Ug)
    first, last = U[:, plan.offsets[:-1]], U[:, plan.offsets[1:] - 1]

    def flux(S):
        rho_, m_, E_ = S
        u_ = m_ / rho_
        p_ = (GAMMA - 1.0) * (E_ - 0.5 * m_ * u_)
        return np.array([m_, m_ * u_ + p_, u_ * (E_ + p_)])

    expect = t / dx * (flux(first) - flux(last))
    scale = seg_sum(np.abs(U)) + np.abs(expect)
    assert np.all(np.abs(after - before - expect) <= 1e-12 * scale)
    # sampled problems against the oracle (its own dt each step)
    rng = np.random.default_rng(4096)
    order = np.argsort(sizes)
    pick = np.concatenate([order[:6], rng.choice(order[6:2000], size=6, replace=False)])
    for p in pick:
        n = int(sizes[p])
        g = grid_of(n, dx[p], 1)
        print(f"[batch 4096] oracle run of problem {p} (n = {n})", flush=True)

        def run(S, seed=None):
            tt = 0.0
            for k in range(100):
                h = CFL / orc.max_wave_speed(S, g, GAMMA)
                S = orc.rk3_step(S, g, 8, 1, 1e-7, GAMMA, h)
                if seed is not None:  # rounding of another evaluation order, every step
                    S = ulp_perturbed(S, seed=seed + 1000 * k)
                tt += h
            return S, tt

        U0 = problem(U, plan, p)
        Uo, to = run(U0)
        # the oracle's own sensitivity to one-ulp differences at every step,
        # over two seeds: the smoothness decisions in nearly flat regions
        # are set by rounding (on any implementation), and over 100 steps
        # such differences can move the state well above one step's rounding
        Up1, _ = run(U0, seed=int(p))
        Up2, _ = run(U0, seed=int(p) + 7)
        spread = np.maximum(np.abs(Up1 - Uo), np.abs(Up2 - Uo))
        tol, _ = conditioning_tol(Uo.T, (Uo + spread).T, field_scale(Uo), factor=8.0)
        err = np.abs(problem(Ug, plan, p) - Uo)
        assert np.all(err <= tol[:, None]), (p, (err / tol[:, None]).max())
        assert t[p] == pytest.approx(to, rel=1e-12)
        left, right = states[p]
        x = W.cell_centres(n, 0.0, 1.0)
        rho_ex, _, _ = ER.sample(left, right, (x - 0.5) / t[p], GAMMA)
        # L1 error in cells, over the exact density's total variation: at
        # most 0.82 on 200 seeded problems of the oracle at n = 256
        l1_cells = np.sum(np.abs(problem(Ug, plan, p)[0] - rho_ex))
        tv = np.sum(np.abs(np.diff(rho_ex)))
        assert l1_cells <= 1.5 * tv, (p, l1_cells, tv)
    plan.close()


# left and right states (rho, u, p) with long constant runs: at rest with signed
# zero momentum, equal on both sides, and states whose flux arithmetic is not
# finite or nearly cancels (a run of those may not be taken for a zero divergence)
FLAT_STATES = [((1.0, 0.0, 1.0), (0.125, -0.0, 0.1)), ((0.5, 0.3, 0.4), (0.5, 0.3, 0.4)),
               ((1.0, 1.0, 1e-9), (1.0, 1.0, 1e-9)), ((1e-120, 0.1, 1e-120), (1e-120, 0.1, 1e-120)),
               ((0.8, -0.9, 0.6), (0.3, 0.7, 0.9))]


@pytest.mark.parametrize("scheme,lim,C_T,bc", [(6, 1, 1e-5, 1), (8, 1, 1e-7, 0), (8, 2, 0.3, 1), (8 | 0x100, 3, 0.0, 1)])
def test_constant_runs_against_the_single_grid_step(T, scheme, lim, C_T, bc):
    """Problems whose segments are constant, partly constant (the jump inside
    the last halo of a segment, at its edges, in its middle) or made of
    extreme constant states: every tile and the persistent launch give the
    bits of the single-grid step by the tile sweep, which has no path for
    constant states, at the step sizes the batch took."""
    sizes, parts = [], []
    for n in (64, 256, 700, 1025):
        for left, right in FLAT_STATES:
            for x0 in (0.5, (n - 3.0) / n, (min(n, 255) + 1.5) / n, 62.0 / n):
                U, _ = W.riemann_problem(n, left, right, gamma=GAMMA, x0=min(x0, 1.0))
                sizes.append(n)
                parts.append(U)
    U = np.concatenate(parts, axis=1)
    dx = 1.0 / np.array(sizes)
    plan = T.BatchPlan(sizes, dx, bc)
    outs = []
    for tile in range(T.BATCH_TILES):
        plan.tile = tile
        outs.append(to_host(plan.rk3(to_dev(U), scheme, lim, C_T, GAMMA, CFL, steps=1)))
    _, dt = plan.times()
    outs.append(to_host(plan.rk3_persistent(to_dev(U), scheme, lim, C_T, GAMMA, CFL, steps=1)))
    T.set_sweep_kernel(T.SWEEP_TILE)
    try:
        for p, n in enumerate(sizes):
            if not np.isfinite(dt[p]):
                continue
            V = to_dev(parts[p])
            T.rk3_step(V, grid_of(n, dx[p], bc), scheme, lim, C_T, GAMMA, dt[p])
            ref = to_host(V)
            for o in outs:
                got = problem(o, plan, p)
                assert np.array_equal(got.view(np.int64), ref.view(np.int64)), (p, n, FLAT_STATES[(p // 4) % 5])
    finally:
        T.set_sweep_kernel(T.SWEEP_AUTO)
    plan.close()


# The sweep of a small batch whose tile nobody chose (one wavefront per field, at
# most 1536 segments of 63 cells; a periodic problem of at most 64 cells is
# one), and batches on both sides of that count.
@pytest.mark.parametrize("sizes", [SIZES + [126, 190, 2000], [63] * 1536, [63] * 1536 + [8]],
                         ids=["ragged", "1536", "1537"])
@pytest.mark.parametrize("scheme,lim,C_T", [(6, 1, 1e-5), (6, 7, 1e-5), (8, 2, 1e-7), (8 | 0x100, 1, 0.0)])
@pytest.mark.parametrize("bc", [0, 1])
def test_small_batches_agree_with_a_chosen_tile(T, sizes, scheme, lim, C_T, bc):
    U, dx, _ = ragged_batch(sizes, seed0=300)
    for p, b in enumerate(np.cumsum([0] + sizes[:-1])):  # the rest flat, extreme or rough
        if p % 3 == 1:
            left, right = FLAT_STATES[(p // 3) % 5]
            U[:, b:b + sizes[p]] = W.riemann_problem(sizes[p], left, right, gamma=GAMMA)[0]
        elif p % 3 == 2:
            U[:, b:b + sizes[p]] *= 1 + 1e-3 * np.random.default_rng(p).standard_normal((3, sizes[p]))
    print(f"[small batch] {len(sizes)} problems {scheme} {lim} bc={bc}", flush=True)
    plan, chosen = T.BatchPlan(sizes, dx, bc), T.BatchPlan(sizes, dx, bc)
    chosen.tile = 3
    assert plan.tile == 3
    want = to_host(chosen.rk3(to_dev(U), scheme, lim, C_T, GAMMA, CFL, steps=2))
    half = len(sizes) // 2
    Ud = to_dev(U)
    plan.rk3(Ud, scheme, lim, C_T, GAMMA, CFL, steps=2, first=0, count=half)
    plan.rk3(Ud, scheme, lim, C_T, GAMMA, CFL, steps=2, first=half)
    Ug = to_dev(U)
    plan.reset_times()
    plan.rk3_graph(Ug, scheme, lim, C_T, GAMMA, CFL, steps=2)
    for got in (to_host(Ud), to_host(Ug)):
        assert np.array_equal(got, want, equal_nan=True)
        finite = np.isfinite(want)
        assert np.array_equal(np.signbit(got[finite]), np.signbit(want[finite]))
    assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(plan.times(), chosen.times()))
    # a tile chosen later takes the tile's kernel, with the same bits
    plan.tile = 0
    Ug = to_dev(U)
    plan.rk3_graph(Ug, scheme, lim, C_T, GAMMA, CFL, steps=2)
    assert np.array_equal(to_host(Ug), want, equal_nan=True)
    plan.close()
    chosen.close()


def test_a_chosen_tile_can_be_undone(T):
    """Setting a tile is seen and can be undone; the automatic choice, the tile and
    the automatic choice again give the same bits, in the captured graph too."""
    sizes = [70, 300, 1000]
    U, dx, _ = ragged_batch(sizes, seed0=40)
    print("[tile reset]", flush=True)
    plan = T.BatchPlan(sizes, dx, 1)
    assert not plan.tile_chosen
    outs = []
    for tile in (None, 5, None):
        if tile is not None:
            plan.tile = tile
        else:
            plan.reset_tile()
        assert plan.tile_chosen == (tile is not None) and plan.tile == (3 if tile is None else tile)
        for call in (plan.rk3, plan.rk3_graph):
            outs.append(to_host(call(to_dev(U), 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=2)))
    assert all(np.array_equal(o, outs[0]) for o in outs)
    plan.close()


@pytest.mark.parametrize("sizes", [[300, 700, 1500, 2000, 900, 600, 2500, 1300], [4000] * 30], ids=["few", "many"])
def test_autotuning_keeps_the_faster_automatic_choice(T, sizes):
    """Few segments: one wavefront per field is a third faster than any tile, so
    autotuning leaves the tile unchosen, whatever was set before; many: a tile is
    chosen.  The reported tile is the fastest of the tiles, and all give the same
    bits."""
    U, dx, _ = ragged_batch(sizes, seed0=41)
    print(f"[autotune] {len(sizes)} problems", flush=True)
    plan, ref = T.BatchPlan(sizes, dx, 1), T.BatchPlan(sizes, dx, 1)
    plan.tile = 4
    Ud = to_dev(U)
    best, ms = plan.autotune(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=20)
    few = sum((n + 62) // 63 for n in sizes) <= 1536
    assert plan.tile == best and ms[best] == min(ms)
    assert plan.tile_chosen == (not few)
    plan.rk3(Ud, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=3)
    want = ref.rk3(to_dev(U), 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=3)
    assert np.array_equal(to_host(Ud), to_host(want))
    # one problem of the batch at a time: the same bits again
    Us = to_dev(U)
    for p in range(len(sizes)):
        plan.rk3(Us, 8, T.LIM_MP, 1e-7, GAMMA, CFL, steps=3, first=p, count=1)
    assert np.array_equal(to_host(Us), to_host(want))
    plan.close()
    ref.close()
