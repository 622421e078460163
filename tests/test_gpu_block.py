"""The block kernel of small grids (WAVE_KERNEL_BLOCK) against the float32
oracle, bit for bit: partial blocks on every axis, layers that are no multiple
of the block, all-layer grids, every storage type and rounding, an eta array,
damping off (both block shapes), sources that share a cell, more sources than
one launch takes, and receivers sampled over several calls."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    from paper_2009_04619_amd import wave
    return wave


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def run(W, shot, calls, kernel, storage="f32", damping=True, sr=False, eta=None):
    sh = W.shot_from_synth(shot, storage=storage, damping=damping, max_steps=sum(calls),
                           stochastic_round=sr, eta=eta)
    sh.set_kernel(*kernel)
    for n in calls:
        sh.step(n)
    out = dict(u=sh.read(W.WAVE_FIELD_U), u_prev=sh.read(W.WAVE_FIELD_UPREV),
               phi=sh.read(W.WAVE_FIELD_PHI), traces=sh.traces())
    sh.close()
    return out


GRIDS = [  # nx, ny, nz, w, storage, damping, sources
    (64, 64, 64, 16, "f32", True, 1),
    (70, 45, 37, 5, "f32", True, 2),
    (129, 17, 22, 7, "bf16", True, 3),
    (200, 37, 13, 3, "f16", True, 4),
    (66, 30, 33, 6, "bf16sr", True, 2),
    (40, 36, 38, 18, "f32", True, 7),        # all layer but a core; more sources than kStepSrc
    (131, 35, 19, 0, "f32", False, 2),
    (65, 33, 11, 0, "f16", False, 5),
    (6, 6, 7, 3, "f32", True, 1),
    (1, 1, 1, 0, "bf16", False, 1),
    (127, 50, 14, 4, "f16", True, 3),        # odd width: the last pair holds a ghost column
    (64, 41, 30, 15, "bf16", True, 6),
]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: f"{g[0]}x{g[1]}x{g[2]}_w{g[3]}_{g[4]}_src{g[6]}")
def test_block_equals_oracle(W, grid):
    nx, ny, nz, w, storage, damping, nsrc = grid
    calls = (1, 6, 2)
    steps = sum(calls)
    shot = synth.config_small_layered(nx, ny, nz, w, steps, seed=nx + 5 * nz, nsrc=nsrc)
    if nsrc > 2:
        shot.src[2] = shot.src[0]           # two sources in one cell, in list order
    expect = oracle.run_shot(shot, steps=steps, precision="f32", storage=storage, damping=damping)
    if not damping:
        expect["phi"] = np.zeros_like(expect["u"])
    sr = storage == "bf16sr"
    kernels = [(10, 1, 4, 4)] + ([] if damping or sr else [(10, 1, 8, 8)]) + \
        ([(10, 1, 8, 4)] if storage in ("bf16", "f16") else [])
    for k in kernels:
        say(f"case block {k} grid {grid}")
        got = run(W, shot, calls, k, "bf16" if sr else storage, damping, sr)
        for key in ("u", "u_prev", "phi", "traces"):
            assert np.array_equal(got[key], expect[key]), (k, grid, key)


def test_block_eta_array(W):
    nx, ny, nz, w = 75, 29, 34, 5
    shot = synth.config_small_layered(nx, ny, nz, w, 8, seed=77, nsrc=2)
    eta = np.random.default_rng(3).uniform(0.0, 0.4, (nz, ny, nx)).astype(np.float32)
    say("case block eta array")
    expect = oracle.run_shot(shot, steps=8, precision="f32", eta=eta)
    got = run(W, shot, (8,), (10, 1, 4, 4), eta=eta)
    for key in ("u", "u_prev", "phi", "traces"):
        assert np.array_equal(got[key], expect[key]), key


def test_block_refusals(W):
    shot = synth.config_small_layered(40, 30, 20, 4, 4, seed=5)
    sh = W.shot_from_synth(shot)
    for bad in ((10, 1, 8, 8), (10, 2, 4, 4), (10, 1, 4, 8), (10, 1, 4, 0), (10, 1, 0, 4), (10, 1, 4, -4),
                (10, 1, 8, 4)):
        assert W.wave_set_kernel(sh.ctx, *bad) == W.WAVE_EINVAL, bad
    assert W.wave_set_kernel(sh.ctx, 10, 1, 4, 4) == W.WAVE_OK
    sh.close()


@pytest.mark.parametrize("storage,kernel", [("f32", (10, 1, 4, 4)), ("bf16", (10, 1, 8, 4))])
def test_block_divisions_over_all_magnitudes(W, storage, kernel):
    """Fields from zero and subnormal to 1e4: the layer's divisions take the
    same bits as the direct kernel's, signs of zeros included."""
    nx, ny, nz, w = 90, 41, 37, 12
    shot = synth.config_small_layered(nx, ny, nz, w, 8, seed=31)
    rng = np.random.default_rng(8)
    state = []
    for _ in range(3):
        # magnitudes vary over blocks, so that whole wavefronts are tiny, mixed or ordinary
        e = rng.uniform(-44.0, 4.0, (nz // 4 + 1, ny // 4 + 1, nx // 30 + 1))
        e = np.kron(e, np.ones((4, 4, 30)))[:nz, :ny, :nx]
        f = rng.standard_normal((nz, ny, nx)) * 10.0 ** e
        f[rng.random((nz, ny, nx)) < 0.02] = 0.0
        f[:, :, 40:60] = -0.0
        state.append(f.astype(np.float32))
    say(f"case block divisions {storage}")
    outs = []
    for k in (kernel, (0, 1, 1, 0)):
        sh = W.shot_from_synth(shot, storage=storage, max_steps=8)
        sh.set_kernel(*k)
        for which, f in zip((W.WAVE_FIELD_U, W.WAVE_FIELD_UPREV, W.WAVE_FIELD_PHI), state):
            sh.write(which, f)
        sh.step(3)
        outs.append([sh.read(i) for i in (W.WAVE_FIELD_U, W.WAVE_FIELD_UPREV, W.WAVE_FIELD_PHI)])
        sh.close()
    for x, y in zip(*outs):
        assert np.isfinite(y).all() and np.array_equal(x.view(np.uint32), y.view(np.uint32))


def _solo(W, args, n):
    sh = _shot(W, *args)
    sh.set_kernel(W.WAVE_KERNEL_DIRECT)
    sh.step(n)
    return _state(W, sh)


def _shot(W, nx, ny, nz, w, nsrc, eta, damping, storage="f32"):
    rng = np.random.default_rng(nx + ny + nsrc)
    vel = rng.uniform(1500.0, 4000.0, (nz, ny, nx)).astype(np.float32)
    e = rng.uniform(0.0, 0.3, (nz, ny, nx)).astype(np.float32) if eta else None
    sh = W.Shot(nx, ny, nz, w, 10.0, 10.0, 10.0, 9e-4, vel, eta=e, damping=damping, storage=storage, max_src=8,
                max_rec=300, max_steps=16)
    for s in range(nsrc):
        p = (nx // 2, ny // 2, nz // 2) if s % 3 == 0 else tuple(int(rng.integers(0, n)) for n in (nx, ny, nz))
        sh.inject(*p, rng.standard_normal(16).astype(np.float32))
    sh.record(np.stack([rng.integers(0, n, 300) for n in (nx, ny, nz)], axis=1))
    return sh


def _state(W, sh):
    out = [sh.read(W.WAVE_FIELD_U), sh.read(W.WAVE_FIELD_UPREV), sh.read(W.WAVE_FIELD_PHI), sh.traces()]
    sh.close()
    return out


# nx, ny, nz, w, sources, eta array, damping
MIXED = [(70, 45, 37, 5, 2, False, True), (64, 30, 40, 4, 1, True, True), (33, 65, 21, 0, 4, False, False),
         (48, 40, 36, 6, 6, False, True),      # more sources than a launch takes: the streaming tile
         (40, 40, 40, 4, 6, True, True), (90, 20, 24, 3, 0, False, True)]
MANY = [(20 + 3 * i, 24, 18 + i, 3, 1, False, True) for i in range(19)]     # more members than a launch holds
LARGE = [(224, 200, 208, 20, 1, False, True)] * 2 + [(64, 64, 64, 8, 1, False, True)]   # more than one group


# 16-bit members on either side of the size where lanes take two points
HALF = [(131, 112, 97, 9, 2, False, True, "bf16"), (128, 120, 90, 0, 1, False, False, "bf16"),
        (60, 44, 30, 4, 3, False, True, "bf16"), (50, 44, 30, 4, 1, True, True, "bf16"),
        (128, 112, 100, 20, 1, False, True, "bf16")]


@pytest.mark.parametrize("graph", [0, 2])
@pytest.mark.parametrize("members", [MIXED, MANY, LARGE, HALF], ids=["mixed", "many", "large", "half"])
def test_batch_by_size_equals_solo(W, members, graph):
    """A batch without a set tile: kinds of sweep side by side, members that
    stop early, runs that continue, several groups."""
    say(f"case batch by size, {len(members)} members, graph {graph}")
    n = [3 + (5 * i) % 7 for i in range(len(members))]
    b = W.Batch(storage=members[0][7] if len(members[0]) > 7 else "f32", max_shots=len(members))
    b.set_graph(graph)
    shots = [_shot(W, *m) for m in members]
    for sh, k in zip(shots, n):
        b.add(sh, k)
    b.run(4)
    b.run(16)
    for sh in shots:
        assert b.remaining(sh) == 0
    b.close()
    for i, sh in enumerate(shots):
        for x, y in zip(_state(W, sh), _solo(W, members[i], n[i])):
            assert x.shape == y.shape and np.array_equal(x, y), (i, members[i])


@pytest.mark.parametrize("nx", [64, 65, 96, 97, 128, 129, 160, 161])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16", "bf16sr"])
def test_block_tile_widths(W, nx, storage):
    """Either side of each change between 64 and 32 columns per block, with
    sources one above the other in both rows of a 32-wide wavefront and in the
    first and last column."""
    ny, nz, w, steps = 27, 15, 4, 5
    shot = synth.config_small_layered(nx, ny, nz, w, steps, seed=nx, nsrc=4)
    for s, p in enumerate(((nx - 1, 12, 7), (nx - 1, 13, 7), (31, 13, 7), (0, 26, 14))):
        shot.src[s] = p
    expect = oracle.run_shot(shot, steps=steps, precision="f32", storage=storage)
    say(f"case block width {nx} {storage}")
    got = run(W, shot, (2, 3), (10, 1, 4, 4), storage.replace("sr", ""), sr=storage == "bf16sr")
    for key in ("u", "u_prev", "phi", "traces"):
        assert np.array_equal(got[key], expect[key]), (nx, storage, key)


# 16-bit members with more sources than a sweep launch takes, among others: damping off,
# tables and an eta array
SOURCES16 = [(100, 40, 30, 4, 6, False, True, "bf16"), (60, 40, 30, 4, 6, False, True, "bf16"),
            (131, 30, 26, 4, 5, False, True, "bf16"), (64, 33, 20, 0, 7, False, False, "bf16"),
            (70, 30, 30, 4, 5, True, True, "bf16"), (200, 24, 22, 4, 5, False, True, "bf16"),
            (50, 30, 30, 4, 2, False, True, "bf16")]


def _member(W, nx, ny, nz, w, nsrc, eta, damping, storage):
    """A member from a random state, `storage` "bf16sr" for stochastic rounding."""
    rng = np.random.default_rng(2 * nx + ny + nsrc)
    vel = rng.uniform(1500.0, 4000.0, (nz, ny, nx)).astype(np.float32)
    e = rng.uniform(0.0, 0.3, (nz, ny, nx)).astype(np.float32) if eta else None
    sh = W.Shot(nx, ny, nz, w, 10.0, 10.0, 10.0, 5e-4, vel, eta=e, damping=damping, storage=storage.replace("sr", ""),
                stochastic_round=storage.endswith("sr"), max_src=8, max_rec=70, max_steps=16)
    for s in range(nsrc):
        p = (nx // 2, ny // 2, nz // 2) if s % 3 == 0 else tuple(int(rng.integers(0, n)) for n in (nx, ny, nz))
        sh.inject(*p, rng.standard_normal(16).astype(np.float32))
    sh.record(np.stack([rng.integers(0, n, 70) for n in (nx, ny, nz)], axis=1))
    for which in (W.WAVE_FIELD_U, W.WAVE_FIELD_UPREV):
        sh.write(which, rng.standard_normal((nz, ny, nx)).astype(np.float32))
    return sh


@pytest.mark.parametrize("graph", [0, 2])
@pytest.mark.parametrize("storage", ["bf16", "f16", "bf16sr"])
def test_batch_of_16_bit_members_with_many_sources(W, storage, graph):
    say(f"case batch by size, 16-bit members with many sources, {storage}, graph {graph}")
    members = [m[:7] + (storage,) for m in SOURCES16]
    n = [3 + (5 * i) % 7 for i in range(len(members))]
    b = W.Batch(storage=storage.replace("sr", ""), max_shots=len(members))
    b.set_graph(graph)
    shots = [_member(W, *m) for m in members]
    for sh, k in zip(shots, n):
        b.add(sh, k)
    for k in (4, 1, 16):
        b.run(k)
    b.close()
    for i, sh in enumerate(shots):
        solo = _member(W, *members[i])
        solo.set_kernel(W.WAVE_KERNEL_DIRECT)
        solo.step(n[i])
        for x, y in zip(_state(W, sh), _state(W, solo)):
            assert np.isfinite(y).all() and np.array_equal(x, y), (i, members[i])


@pytest.mark.parametrize("members", [MIXED, MANY, LARGE, HALF], ids=["mixed", "many", "large", "half"])
def test_batch_runs_of_one_step(W, members):
    """Runs of one step, which launch more members together than longer ones and add
    sources and sample receivers apart, between longer ones; members that have ended
    lie between those that have not."""
    say(f"case batch one step a run, {len(members)} members")
    n = [3 + (5 * i) % 7 for i in range(len(members))]
    b = W.Batch(storage=members[0][7] if len(members[0]) > 7 else "f32", max_shots=len(members))
    shots = [_shot(W, *m) for m in members]
    for sh, k in zip(shots, n):
        b.add(sh, k)
    for k in (1, 1, 2, 1, 3, 1, 1, 1):
        b.run(k)
    for sh in shots:
        assert b.remaining(sh) == 0
    b.close()
    for i, sh in enumerate(shots):
        for x, y in zip(_state(W, sh), _solo(W, members[i], n[i])):
            assert x.shape == y.shape and np.array_equal(x, y), (i, members[i])


# few rows of blocks, which XCDs take in runs: 1 to 7, 9 and 10 tile rows of 4 and of 8,
# with the last run ending in, at and past the last row
THIN = [(70, 3, 40, 1, "f32", True), (66, 5, 21, 2, "f32", True), (130, 9, 33, 3, "bf16", True),
        (65, 17, 26, 5, "f16", True), (200, 20, 18, 4, "f32", True), (90, 33, 25, 8, "bf16sr", True),
        (64, 36, 30, 3, "f32", True), (129, 40, 22, 6, "bf16", True), (64, 72, 19, 5, "f16", True),
        (70, 5, 41, 0, "f32", False), (66, 9, 65, 0, "bf16", False), (40, 72, 9, 0, "f32", False),
        (33, 1, 50, 0, "f16", False), (1, 2, 9, 0, "f32", False)]


def _run_state(W, grid, kernel, steps, dt=2e-4, eta=False):
    """Fields and traces after `steps` from a random state, under `kernel`."""
    nx, ny, nz, w, storage, damping = grid
    rng = np.random.default_rng(nx + 3 * ny + nz)
    vel = rng.uniform(1500.0, 4000.0, (nz, ny, nx)).astype(np.float32)
    e = rng.uniform(0.0, 0.3, (nz, ny, nx)).astype(np.float32) if eta else None
    sh = W.Shot(nx, ny, nz, w, 10.0, 10.0, 10.0, dt, vel, eta=e, damping=damping, max_src=2, max_rec=90, max_steps=16,
                storage=storage.replace("sr", ""), stochastic_round=storage.endswith("sr"))
    for p in ((nx - 1, ny - 1, nz - 1), (nx // 2, ny // 2, nz // 2)):
        sh.inject(*p, rng.standard_normal(16).astype(np.float32))
    sh.record(np.stack([rng.integers(0, n, 90) for n in (nx, ny, nz)], axis=1))
    for which in [W.WAVE_FIELD_U, W.WAVE_FIELD_UPREV] + ([W.WAVE_FIELD_PHI] if damping else []):
        sh.write(which, rng.standard_normal((nz, ny, nx)).astype(np.float32))
    if kernel:
        sh.set_kernel(*kernel)
    for n in steps:
        sh.step(n)
    return _state(W, sh)


@pytest.mark.parametrize("grid", THIN, ids=lambda g: f"{g[0]}x{g[1]}x{g[2]}_w{g[3]}_{g[4]}")
def test_thin_grids(W, grid):
    storage, damping = grid[4:]
    sr = storage == "bf16sr"
    expect = _run_state(W, grid, (0, 1, 1, 0), (5,))
    kernels = [(10, 1, 4, 4)] + ([] if damping or sr else [(10, 1, 8, 8)]) + \
        ([(10, 1, 8, 4)] if storage in ("bf16", "f16") else [])
    for k in kernels:
        say(f"case block thin {k} grid {grid}")
        for x, y in zip(_run_state(W, grid, k, (2, 3)), expect):
            assert np.isfinite(y).all() and np.array_equal(x, y), (k, grid)


@pytest.mark.parametrize("nx", [1, 9, 31, 32, 33])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16", "bf16sr"])
def test_narrow_grids(W, nx, storage):
    """Grids one block of 32 columns wide, either side of the count of rows from which
    blocks take them, with a layer, without, and with an eta array."""
    w = min(4, nx // 2)
    for ny, nz in ((64, 64), (63, 65), (37, 150)):
        for damping, eta in ((True, False), (False, False), (True, True)):
            if w == 0 and damping:
                continue
            say(f"case narrow {nx}x{ny}x{nz} {storage} damping {damping} eta {eta}")
            grid = (nx, ny, nz, w if damping else 0, storage, damping)
            got, expect = (_run_state(W, grid, k, (2, 1), eta=eta) for k in ((10, 1, 4, 4), (0, 1, 1, 0)))
            for x, y in zip(got, expect):
                assert np.isfinite(y).all() and np.array_equal(x, y), grid
