"""The tile sweep against the line sweeps and the oracle, on every axis.

The tile sweep (a workgroup stages tiles of 8 adjacent lines by a chunk of
the line in LDS and walks the lines whole, handing each chunk's last face to
the next; the lines are x columns for y and z, y rows for x) and the line
kernels (the row sweep for x; for y and z the march, one lane per x column
with its stencil in an LDS ring) evaluate the same face fluxes and cell
updates operation for operation, so their results must agree bit for bit.
The shapes put line lengths below, at and just above one chunk (32 faces)
and several chunks with a ragged last one, on every axis, extents across
the lines that leave part of the last group of 8 outside the grid, and both
boundary rules on every axis; the automatic choice takes the line kernels
for all of them, so each kernel is forced through tenom_set_sweep_kernel.
One case per scheme also goes to the oracle on the tile path directly
(1e-12 of each field's largest magnitude outside the cutoff band, as in the
other parity tests).
"""
import numpy as np
import pytest

import workloads as W
from parity import assert_close_fields, require_gpu, to_dev, to_host
from test_gpu_parity import CASES, make, rk3_band_cells

pytestmark = pytest.mark.gpu

GAMMA = 1.4

# name, shape (z, y, x order), bc (x, y, z order), scheme, limiter, C_T
SHAPES = [
    ("chunk_below", (20, 31, 13), [0, 0, 1], 6, 1, 1e-5),
    ("chunk_exact", (32, 32, 16), [1, 0, 0], 6, 1, 1e-5),
    ("chunk_above", (33, 33, 9), [0, 1, 0], 8, 1, 1e-7),
    ("chunks_ragged", (70, 12, 24), [0, 0, 0], 6, 3, 1e-5),
    ("chunks_ragged_trans", (12, 97, 17), [1, 1, 1], 8, 2, 1e-7),
    ("two_chunks_exact", (64, 9, 8), [0, 1, 1], 8 | 0x100, 1, 0.0),
    ("narrow_x", (40, 36, 6), [0, 0, 1], 6, 7, 1e-5),
    ("teno8_long_y", (9, 129, 11), [1, 0, 0], 8, 0, 1e-6),
    ("x_chunks_ragged", (6, 13, 70), [0, 1, 0], 6, 1, 1e-5),
    ("x_two_chunks_exact", (8, 17, 64), [1, 0, 0], 8, 1, 1e-7),
    ("x_chunk_above", (8, 8, 33), [0, 0, 1], 8 | 0x100, 1, 0.0),
]
SHAPE_IDS = [s[0] for s in SHAPES]
MULTI_D = [c for c in CASES if len(c[1]) >= 2]


@pytest.fixture(scope="module")
def T():
    require_gpu()
    import paper_2010_13289_amd as T
    yield T
    T.set_sweep_kernel(T.SWEEP_AUTO)


def both_kernels(T, fn):
    out = []
    for kind in (T.SWEEP_TILE, T.SWEEP_MARCH):
        T.set_sweep_kernel(kind)
        out.append(fn())
    T.set_sweep_kernel(T.SWEEP_AUTO)
    return out


def shape_case(spec, seed):
    name, shape, bc, K, lim, C_T = spec
    n = list(reversed(shape))
    grid = dict(ndim=3, n=n, dx=[0.05, 0.07, 0.06], bc=bc, system=1)
    U = W.random_euler_state(shape, seed=seed, kind="mixed")
    return grid, U, K, lim, C_T


def check_identical(T, grid, U, K, lim, C_T, what):
    dt = 0.4 / T.max_wave_speed(to_dev(U), grid, GAMMA)

    def div():
        return to_host(T.flux_divergence(to_dev(U), grid, K, lim, C_T, GAMMA))

    def step():
        Ud = to_dev(U)
        T.rk3_step(Ud, grid, K, lim, C_T, GAMMA, dt)
        return to_host(Ud)

    d_tile, d_march = both_kernels(T, div)
    assert np.array_equal(d_tile, d_march), f"{what}: divergence differs between the sweep kernels"
    s_tile, s_march = both_kernels(T, step)
    assert np.array_equal(s_tile, s_march), f"{what}: RK3 step differs between the sweep kernels"
    return d_tile, s_tile, dt


@pytest.mark.parametrize("spec", SHAPES, ids=SHAPE_IDS)
def test_tile_and_march_agree_on_chunk_shapes(T, spec):
    grid, U, K, lim, C_T = shape_case(spec, seed=31)
    print(f"[sweep kernels] {spec[0]} n={grid['n']} bc={grid['bc']}", flush=True)
    check_identical(T, grid, U, K, lim, C_T, spec[0])


@pytest.mark.parametrize("case", MULTI_D, ids=[c[0] for c in MULTI_D])
def test_tile_and_march_agree_on_parity_cases(T, case):
    grid, U, K, lim, C_T = make(case, seed=5)
    print(f"[sweep kernels] {case[0]}", flush=True)
    check_identical(T, grid, U, K, lim, C_T, case[0])


ORACLE_SHAPES = [SHAPES[i] for i in (1, 4, 5, 8)]


@pytest.mark.parametrize("spec", ORACLE_SHAPES, ids=[s[0] for s in ORACLE_SHAPES])
def test_tile_against_the_oracle(T, orc, spec):
    grid, U, K, lim, C_T = shape_case(spec, seed=43)
    print(f"[tile vs oracle] {spec[0]}", flush=True)
    T.set_sweep_kernel(T.SWEEP_TILE)
    try:
        dt = 0.4 / orc.max_wave_speed(U, grid, GAMMA)
        Ud = to_dev(U)
        T.rk3_step(Ud, grid, K, lim, C_T, GAMMA, dt)
        Ug = to_host(Ud)
    finally:
        T.set_sweep_kernel(T.SWEEP_AUTO)
    Uo = orc.rk3_step(U, grid, K, lim, C_T, GAMMA, dt)
    excl = rk3_band_cells(orc, U, grid, K, lim, C_T, dt)
    assert_close_fields(Ug, Uo, exclude=excl, what=f"{spec[0]} RK3 step, tile sweeps")


def test_automatic_choice_at_64_cubed_against_the_oracle(T, orc):
    """At 64^3 the lines of every axis give 512 tile workgroups, so the
    automatic choice runs the tile sweeps: the divergence of a seeded state against
    the oracle over every cell outside the cutoff band (1e-12 of each field's
    largest magnitude)."""
    from parity import band_faces, faces_to_cells
    shape = (64, 64, 64)
    grid = dict(ndim=3, n=[64, 64, 64], dx=[0.05, 0.07, 0.06], bc=[0, 1, 0], system=1)
    U = W.random_euler_state(shape, seed=57, kind="mixed")
    K, lim, C_T = 6, 1, 1e-5
    print("[automatic choice] 64^3 divergence", flush=True)
    T.set_sweep_kernel(T.SWEEP_AUTO)
    dg = to_host(T.flux_divergence(to_dev(U), grid, K, lim, C_T, GAMMA))
    do = orc.flux_divergence(U, grid, K, lim, C_T, GAMMA)
    excl = np.zeros(shape, dtype=bool)
    for axis in range(3):
        _, _, bd = orc.reconstruct_faces(U, grid, K, lim, C_T, GAMMA, axis)
        excl |= faces_to_cells(band_faces(bd), 2 - axis, 64, grid["bc"][axis] == 0, 1)
    assert excl.mean() < 0.01
    assert_close_fields(dg, do, exclude=excl, what="64^3 dU/dt, automatic sweep kernels")


# Line lengths at the edges of the one-chunk segments that small grids take
# (31 cells; a periodic line of at most 32 wraps whole), in 2D; then grids with
# enough lines for segments of several chunks and for whole lines, each along
# x (with the periodic walk's shifted start) and a strided axis.
SEGMENT_SHAPES = [((m, 9), [b, 1 - b], K) for m in (31, 32, 33, 62, 63, 64, 94) for b in (0, 1) for K in (6, 8)]
SEGMENT_SHAPES += [((9, m), [b, 0], 6) for m in (32, 33, 63) for b in (0, 1)]
SEGMENT_SHAPES += [((70, 160, 200), [0, 0, 0], 6), ((200, 160, 70), [0, 1, 1], 6), ((150, 93, 187), [1, 0, 0], 8),
                   ((136, 128, 100), [0, 1, 1], 8)]


@pytest.mark.parametrize("shape,bc,K", SEGMENT_SHAPES, ids=[f"{'x'.join(map(str, s))}-{''.join(map(str, b))}-{k}"
                                                            for s, b, k in SEGMENT_SHAPES])
def test_segments_agree_with_the_march(T, shape, bc, K):
    n = list(reversed(shape))
    grid = dict(ndim=len(n), n=n, dx=[0.05, 0.07, 0.06][:len(n)], bc=bc, system=1)
    U = W.random_euler_state(shape, seed=sum(shape) + K, kind="mixed")
    print(f"[segments] n={n} bc={bc} K={K}", flush=True)
    check_identical(T, grid, U, K, 1, 1e-5 if K == 6 else 1e-7, "segments")


# 1D lines, where the automatic choice takes a whole step in one launch (up to
# 256 faces of the Euler equations, 1024 of the scalar equation) and, above,
# sweeps with one wavefront per field (workgroups of 63 cells, or a periodic
# line of at most 64 whole), against the row sweep that the line setting
# forces.  A periodic line has n faces, a transmissive one n + 1.
LINES = [(n, bc, 1, K, lim) for n, K, lim in ((8, 8, 0), (63, 6, 1), (64, 8, 2), (65, 6, 3), (127, 8 | 0x100, 1),
                                               (255, 6, 7), (256, 8, 1), (257, 8, 3), (378, 6, 0), (1001, 8 | 0x100, 2),
                                               (40960, 6, 1), (40961, 8, 1)) for bc in (0, 1)]
LINES += [(n, bc, 0, K, lim) for n, K, lim in ((6, 6, 0), (65, 8, 1), (200, 6, 1), (1023, 8 | 0x100, 2), (1024, 6, 3),
                                               (1025, 8, 1)) for bc in (0, 1)]


def line_case(n, bc, system, seed):
    grid = dict(ndim=1, n=[n], dx=[1.0 / n], bc=[bc], system=system, adv=[-0.7, 0.0, 0.0])
    if system == 1:
        return grid, W.random_euler_state((n,), seed=seed, kind="mixed")
    x = (np.arange(n) + 0.5) / n
    U = np.sin(2 * np.pi * x) + (np.abs(x - 0.5) < 0.2) + 1e-3 * np.random.default_rng(seed).standard_normal(n)
    return grid, U[None]


@pytest.mark.parametrize("n,bc,system,K,lim", LINES, ids=["-".join(map(str, c)) for c in LINES])
def test_line_kernels_agree_with_the_row_sweep(T, n, bc, system, K, lim):
    import torch
    C_T = 0.0 if K & 0x100 else (1e-5 if K == 6 else 1e-7)
    grid, U = line_case(n, bc, system, seed=n + K)
    print(f"[lines] n={n} bc={bc} system={system} K={K} lim={lim}", flush=True)
    dt = 0.4 / T.max_wave_speed(to_dev(U), grid, GAMMA)

    def results():
        Ud = to_dev(U)
        out = [to_host(T.flux_divergence(Ud, grid, K, lim, C_T, GAMMA))]
        T.rk3_step(Ud, grid, K, lim, C_T, GAMMA, dt)
        out.append(to_host(Ud))
        dts = torch.zeros(1, dtype=torch.float64, device="cuda")
        for _ in range(2):
            T.rk3_step_cfl(Ud, grid, K, lim, C_T, GAMMA, 0.4, dt_out=dts)
            out += [to_host(Ud), dts.cpu().numpy()]
        return out

    got = {}
    for kind in (T.SWEEP_AUTO, T.SWEEP_MARCH):
        T.set_sweep_kernel(kind)
        try:
            got[kind] = results()
        finally:
            T.set_sweep_kernel(T.SWEEP_AUTO)
    names = ("divergence", "RK3 step", "CFL step", "dt", "second CFL step", "second dt")
    for name, a, b in zip(names, got[T.SWEEP_AUTO], got[T.SWEEP_MARCH]):
        assert np.array_equal(a, b), f"{name} differs between the line kernels and the row sweep"


@pytest.mark.parametrize("n,system", [(200, 1), (500, 1), (300, 0)])
def test_line_steps_in_a_captured_graph(T, n, system):
    """Three CFL steps captured once and replayed, with eager steps of another
    state and a synchronisation between the replays: the eager result, bit for
    bit, after each."""
    import torch
    grid, U = line_case(n, 0, system, seed=n)
    args = (grid, 6, 1, 1e-5, GAMMA, 0.4)
    print(f"[line graph] n={n} system={system}", flush=True)
    Ug, Ue, other = to_dev(U), to_dev(U), to_dev(U)
    wsg, wse = T.Workspace(grid, 6), T.Workspace(grid, 6)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        T.rk3_step_cfl(other, *args, workspace=wsg, stream=side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(3):
            T.rk3_step_cfl(Ug, *args, workspace=wsg, stream=side)
    for replay in range(3):
        graph.replay()
        T.rk3_step_cfl(other, *args, workspace=wse)
        for _ in range(3):
            T.rk3_step_cfl(Ue, *args, workspace=wse)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(Ug), to_host(Ue)), f"replay {replay}"


# Face fluxes of grids small enough for one wavefront per field (NF wavefronts of
# 64 faces, at most 4096 in all: 8 lines by 8 faces; 64 of a single line) against
# the same cells repeated along another axis until the grid takes the other face
# kernel; in 1D against the row sweep's divergence.  z, y, x order; the repeated
# axis is the first that is not the face's.
SMALL_FACES = [((m, 8), [b, 1 - b], K) for m in (8, 9, 15, 17) for b in (0, 1) for K in (6, 8, 8 | 0x100)]
SMALL_FACES += [((9, 23, 8), [0, 1, 0], 6), ((8, 9, 17), [1, 0, 1], 8), ((12, 8, 9), [0, 0, 0], 8 | 0x100)]


@pytest.mark.parametrize("lim", [1, 2])
@pytest.mark.parametrize("shape,bc,K", SMALL_FACES, ids=[f"{'x'.join(map(str, s))}-{''.join(map(str, b))}-{k}"
                                                         for s, b, k in SMALL_FACES])
def test_small_faces_agree_with_repeated_cells(T, shape, bc, K, lim):
    C_T = 0.0 if K & 0x100 else (1e-5 if K == 6 else 1e-7)
    nd = len(shape)
    U = W.random_euler_state(shape, seed=sum(shape) + K, kind="mixed")
    print(f"[small faces] {shape} {bc} {K}", flush=True)
    for axis in range(nd):
        along = nd - 1 - axis  # the face's axis among z, y, x
        other = next(a for a in range(nd) if a != along)
        copies = 1 + (4096 * 64) // int(np.prod(shape))
        big = list(shape)
        big[other] *= copies
        out = []
        for s, V in ((shape, U), (tuple(big), np.concatenate([U] * copies, axis=1 + other))):
            grid = dict(ndim=nd, n=list(reversed(s)), dx=[0.05, 0.07, 0.06][:nd], bc=bc, system=1)
            for flags in (False, True):
                r = T.reconstruct_faces(to_dev(V), grid, K, lim, C_T, GAMMA, axis, return_flags=flags)
                out.append([to_host(x) for x in r] if flags else [to_host(r)])
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[2][0], out[3][0])
        for k, small, large in ((0, out[1][0], out[3][0]), (1, out[1][1], out[3][1])):
            ax = small.ndim - nd + other
            for piece in np.split(large, copies, axis=ax):
                assert np.array_equal(piece, small), (axis, "flux" if k == 0 else "flags")


@pytest.mark.parametrize("n", [8, 63, 64, 65, 128, 87360, 87424])
@pytest.mark.parametrize("bc", [0, 1])
def test_line_faces_agree_with_the_row_sweep(T, n, bc):
    grid, U = line_case(n, bc, 1, seed=n)
    print(f"[line faces] {n} {bc}", flush=True)
    for K, lim in ((6, 1), (8, 3)):
        F = T.reconstruct_faces(to_dev(U), grid, K, lim, 1e-5, GAMMA, 0)
        F = to_host(F[0] if isinstance(F, tuple) else F)
        T.set_sweep_kernel(T.SWEEP_MARCH)
        try:
            D = to_host(T.flux_divergence(to_dev(U), grid, K, lim, 1e-5, GAMMA))
        finally:
            T.set_sweep_kernel(T.SWEEP_AUTO)
        assert np.array_equal((F[:, :-1] - F[:, 1:]) * (1.0 / grid["dx"][0]), D)


# Face fluxes of grids above the one-wavefront-per-field kernel, whose lines the
# 32-face chunks of 8 lines fill badly (whole short lines, or equal chunks of many
# lines, side by side) or well: the fluxes along an axis do not depend on the
# other axes' extents, so blocks of lines taken as grids of their own (the other
# kernel) give the same bits.  z, y, x order.
FACE_SPLITS = [((12, 100, 101), 6, 1), ((50, 49, 50), 8, 1), ((33, 72, 73), 8 | 0x100, 3), ((33, 72, 73), 6, 2),
               ((64, 64, 61), 8, 4), ((7, 160, 201), 6, 1), ((300, 401), 8, 1), ((1394, 130), 6, 7), ((8, 20000), 8, 2)]


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("shape,K,lim", FACE_SPLITS, ids=["x".join(map(str, c[0])) + f"-{c[1]}-{c[2]}" for c in FACE_SPLITS])
def test_face_splits_agree_with_blocks_of_lines(T, shape, K, lim, bc):
    C_T = 0.0 if K & 0x100 else (1e-5 if K == 6 else 1e-7)
    nd = len(shape)
    U = W.random_euler_state(shape, seed=sum(shape) + K, kind="mixed")
    print(f"[face split] {shape} {K} {lim} bc={bc}", flush=True)

    def faces(V, axis):
        grid = dict(ndim=nd, n=list(reversed(V.shape[1:])), dx=[0.05, 0.07, 0.06][:nd], bc=[bc] * nd, system=1)
        return [to_host(a) for a in T.reconstruct_faces(to_dev(V), grid, K, lim, C_T, GAMMA, axis, return_flags=True)]

    for axis in range(nd):
        along = nd - 1 - axis
        whole = faces(U, axis)
        across = [a for a in range(nd) if a != along]
        # blocks of at most 16 x 16 lines in 3D, 24 in 2D; the first, a middle and the last
        step = 16 if nd == 3 else 24
        starts = [sorted({0, max(0, (shape[a] // step // 2) * step), max(0, shape[a] - step)}) for a in across]
        for at in np.ndindex(*[len(s) for s in starts]):
            cut = [slice(None)] * (nd + 1)
            for a, s, i in zip(across, starts, at):
                cut[1 + a] = slice(s[i], s[i] + step)
            part = faces(np.ascontiguousarray(U[tuple(cut)]), axis)
            assert np.array_equal(part[0], whole[0][tuple(cut)]), (axis, at, "flux")
            assert np.array_equal(part[1], whole[1][(slice(None),) + tuple(cut)]), (axis, at, "flags")


def test_faces_of_the_most_short_lines(T):
    """300 million scalar lines of 7 cells: a launch of chunks of 32 faces each
    would have more than 2^32 threads."""
    import torch
    nx, ny, nz = 32768, 9300, 7
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    print(f"[many lines] {nx}x{ny}x{nz}", flush=True)
    U = torch.empty((1, nz, ny, nx), dtype=torch.float64, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    for z in range(nz):
        U[0, z].uniform_(-1.0, 1.0, generator=gen)

    def grid(V):
        return dict(ndim=3, n=list(reversed(V.shape[1:])), dx=[0.1] * 3, bc=[0, 0, 0], system=0, adv=[0.3, -0.2, 0.7])

    F = T.reconstruct_faces(U, grid(U), 6, 1, 1e-5, GAMMA, 2)
    F = F[0] if isinstance(F, tuple) else F
    for y in (0, 4095, 8191, ny - 16):
        for x in (0, 16000, nx - 64):
            V = U[:, :, y:y + 16, x:x + 64].contiguous()
            f = T.reconstruct_faces(V, grid(V), 6, 1, 1e-5, GAMMA, 2)
            f = f[0] if isinstance(f, tuple) else f
            assert torch.equal(f, F[:, :, y:y + 16, x:x + 64]), (y, x)
    del U, F
    torch.cuda.empty_cache()


# Grids whose faces run straight from global memory on some axis: just above the
# one-wavefront-per-field kernel, on both sides of 65,536 and of 131,072 faces.
DIRECT_FACES = [((39, 40, 40), 6, 3), ((40, 39, 40), 8 | 0x100, 1), ((250, 259), 8, 2), ((256, 257), 6, 4),
                ((32, 41, 50), 6, 0), ((50, 51, 50), 6, 6), ((50, 49, 51), 8, 8), ((13, 94, 100), 8 | 0x100, 3)]


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("shape,K,lim", DIRECT_FACES, ids=["x".join(map(str, c[0])) + f"-{c[1]}-{c[2]}" for c in DIRECT_FACES])
def test_direct_faces_agree_with_blocks_of_lines(T, shape, K, lim, bc):
    test_face_splits_agree_with_blocks_of_lines(T, shape, K, lim, bc)


# Runs of one state whose faces are not finite (negative pressure, vacuum, NaN,
# overflow) or extreme, with a cutoff that no constant stencil passes: a long line,
# whose wavefronts take constant states at once, against a short one, which does
# not look for them.
@pytest.mark.parametrize("K,lim,C_T", [(8, 1, 0.3), (6, 2, 0.3), (6, 7, 1e-5), (8 | 0x100, 3, 0.0)])
def test_faces_of_constant_lines_that_are_not_finite(T, K, lim, C_T):
    states = [(1.0, 0.0, -1.0), (1.0, -1.0, 0.2), (0.0, 0.0, 1.0), (np.nan, 0.0, 1.0), (1.0, np.nan, 1.0),
              (1.0, 0.5, np.inf), (1e290, 1e293, 5.0000001e295), (1.0, 1e120, 1e240), (1e-300, 0.0, 1e10), (1.0, 0.3, 2.0)]
    print(f"[constant line] {K} {lim} {C_T}", flush=True)
    for state in states:
        out = []
        for n in (88, 90112):
            grid = dict(ndim=1, n=[n], dx=[0.1], bc=[0], system=1)
            U = np.repeat(np.array(state)[:, None], n, axis=1)
            F, flags = T.reconstruct_faces(to_dev(U), grid, K, lim, C_T, GAMMA, 0, return_flags=True)
            out.append((to_host(F), to_host(flags)))
        (F0, f0), (F1, f1) = out
        assert np.array_equal(np.broadcast_to(F0[:, :1], F1.shape), F1, equal_nan=True), state
        assert np.array_equal(np.broadcast_to(f0[:, :, :1], f1.shape), f1), state
