"""Default paths of the block kernel and of batches that the tests of their own
files do not reach, bit for bit against the direct kernel or solo runs: blocks that
go around the memory-side cache, stochastic rounding in batches, divisions over all
magnitudes in every block shape and with an eta array, overflow to infinity and NaN,
and the streaming batch path (graph replays over several runs, membership, another
stream), which batches take under a set tile."""
import sys

import numpy as np
import pytest


pytestmark = pytest.mark.gpu
DIRECT = (0, 1, 1, 0)


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


def make(W, nx, ny, nz, w, storage, damping=True, eta=False, nsrc=2, seed=0, dt=5e-4, state=None, stream=None):
    """A shot, its state random unless given; storage "bf16sr": stochastic rounding."""
    rng = np.random.default_rng(nx + 3 * ny + nz + seed)
    vel = np.resize(rng.uniform(1500.0, 4000.0, 65537).astype(np.float32), (nz, ny, nx))
    e = rng.uniform(0.0, 0.3, (nz, ny, nx)).astype(np.float32) if eta else None
    sh = W.Shot(nx, ny, nz, w, 10.0, 10.0, 10.0, dt, vel, eta=e, damping=damping, storage=storage.replace("sr", ""),
                stochastic_round=storage.endswith("sr"), max_src=8, max_rec=40, max_steps=48, stream=stream)
    for s in range(nsrc):
        p = (nx // 2, ny // 2, nz // 2) if s % 3 == 0 else tuple(int(rng.integers(0, n)) for n in (nx, ny, nz))
        sh.inject(*p, rng.standard_normal(48).astype(np.float32))
    sh.record(np.stack([rng.integers(0, n, 40) for n in (nx, ny, nz)], axis=1))
    fields = [W.WAVE_FIELD_U, W.WAVE_FIELD_UPREV] + ([W.WAVE_FIELD_PHI] if damping else [])
    if state is None:
        base = rng.standard_normal(131071).astype(np.float32)
        state = [np.resize(np.roll(base, 1000 * q), (nz, ny, nx)) for q in range(3)]
    for which, f in zip(fields, state):
        sh.write(which, f)
    return sh


def end(W, sh, close=True):
    out = [sh.read(W.WAVE_FIELD_U), sh.read(W.WAVE_FIELD_UPREV), sh.read(W.WAVE_FIELD_PHI), sh.traces()]
    if close:
        sh.close()
    return out


def same(got, want, what):
    for q, (x, y) in enumerate(zip(got, want)):
        assert x.shape == y.shape and np.array_equal(x, y), (what, q)


def bits_same(got, want, what):
    """The same bits, signs of zeros included; NaN wherever the other has one."""
    for q, (x, y) in enumerate(zip(got, want)):
        x, y = np.asarray(x, np.float32), np.asarray(y, np.float32)
        nan = np.isnan(y)
        assert np.array_equal(np.isnan(x), nan), (what, q, "NaN")
        assert np.array_equal(x.view(np.uint32)[~nan], y.view(np.uint32)[~nan]), (what, q)


@pytest.mark.parametrize("grid,storage", [((333, 317, 321), "f32"), ((379, 371, 367), "bf16"), ((379, 371, 367), "f16")])
def test_blocks_around_the_cache(W, grid, storage):
    """Past 400 MB of state and without a layer, the default (8 x 8 x 8 blocks, all but
    u^n around the memory-side cache): two steps from a random state, the extents
    partial blocks on every axis."""
    say(f"case no layer, {grid} {storage}")
    shots = [make(W, *grid, 0, storage, damping=False) for _ in range(2)]
    shots[1].set_kernel(*DIRECT)
    for sh in shots:
        sh.step(2)
    same(end(W, shots[0]), end(W, shots[1]), storage)


MEMBERS = [(131, 60, 47, 9, True, 2), (128, 50, 40, 0, False, 1), (60, 44, 30, 4, True, 3), (96, 40, 30, 5, True, 1),
           (33, 40, 36, 6, True, 4), (30, 70, 64, 0, False, 2), (64, 36, 30, 4, True, 0)]


@pytest.mark.parametrize("storage", ["bf16sr", "f32", "bf16", "f16"])
def test_batch_of_block_members(W, storage):
    """Members of a kind in one launch, 64 and 32 columns wide, in runs of one step and
    more, stochastic rounding among them."""
    say(f"case batch of block members {storage}")
    for eta in (False, True):
        specs = [m for m in MEMBERS if m[4] or not eta]
        n = [4 + (3 * i) % 7 for i in range(len(specs))]
        b = W.Batch(storage=storage.replace("sr", ""), max_shots=len(specs))
        shots = [make(W, *m[:4], storage, m[4], eta and m[4], m[5], seed=i) for i, m in enumerate(specs)]
        for sh, k in zip(shots, n):
            b.add(sh, k)
        for k in (2, 1, 3, 1, 20):
            b.run(k)
        b.close()
        for i, (m, sh) in enumerate(zip(specs, shots)):
            solo = make(W, *m[:4], storage, m[4], eta and m[4], m[5], seed=i)
            solo.set_kernel(*DIRECT)
            solo.step(n[i])
            same(end(W, sh), end(W, solo), (storage, eta, i))


def magnitudes(nx, ny, nz, lo, hi):
    """Three fields whose magnitudes vary over blocks, so that whole wavefronts are tiny,
    mixed or ordinary, with zeros of both signs."""
    rng = np.random.default_rng(8)
    out = []
    for _ in range(3):
        e = np.kron(rng.uniform(lo, hi, (nz // 4 + 1, ny // 4 + 1, nx // 30 + 1)), np.ones((4, 4, 30)))
        f = rng.standard_normal((nz, ny, nx)) * 10.0 ** e[:nz, :ny, :nx]
        f[rng.random((nz, ny, nx)) < 0.02] = 0.0
        f[:, :, 40:60] = -0.0
        out.append(f.astype(np.float32))
    return out


@pytest.mark.parametrize("nx", [90, 120])      # 32 and 64 columns per block
@pytest.mark.parametrize("eta", [False, True])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16", "bf16sr"])
def test_divisions_over_all_magnitudes(W, storage, eta, nx):
    say(f"case divisions {storage} eta {eta} nx {nx}")
    state = magnitudes(nx, 41, 37, -44.0, 2.0 if storage == "f16" else 4.0)
    kernels = [(10, 1, 4, 4)] + ([(10, 1, 8, 4)] if storage in ("bf16", "f16") and not eta else [])
    outs = []
    for k in [DIRECT] + kernels:
        sh = make(W, nx, 41, 37, 12, storage, True, eta, 0, state=state)
        sh.set_kernel(*k)
        sh.step(3)
        outs.append(end(W, sh))
    assert all(np.isfinite(f).all() for f in outs[0])
    for k, got in zip(kernels, outs[1:]):
        bits_same(got, outs[0], (k, storage, eta))


@pytest.mark.parametrize("nx", [90, 120])
@pytest.mark.parametrize("eta", [False, True])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16", "bf16sr"])
def test_overflow(W, storage, eta, nx):
    """Values near the largest of the storage type in some blocks: infinities and NaN
    come where the direct kernel has them."""
    say(f"case overflow {storage} eta {eta} nx {nx}")
    top = 65504.0 if storage == "f16" else 3e38
    state = magnitudes(nx, 41, 37, -3.0, 2.0)
    for q, f in enumerate(state):
        f[4:9, 8:14, 10:30] = top * (-1) ** q
        f[20:24, 30:33, 64:80] = top / 3
        f[30:, :5, :] *= np.float32(top / 1e6)
    kernels = [(10, 1, 4, 4)] + ([(10, 1, 8, 4)] if storage in ("bf16", "f16") and not eta else [])
    outs = []
    for k in [DIRECT] + kernels:
        sh = make(W, nx, 41, 37, 12, storage, True, eta, 0, state=state)
        sh.set_kernel(*k)
        sh.step(3)
        outs.append(end(W, sh))
    assert not all(np.isfinite(f).all() for f in outs[0])
    for k, got in zip(kernels, outs[1:]):
        bits_same(got, outs[0], (k, storage, eta))


SMALL = [(70, 45, 37, 5), (128, 48, 64, 8), (33, 90, 41, 4), (200, 24, 22, 4)]


def solo_steps(W, i, storage, n):
    sh = make(W, *SMALL[i], storage, seed=i)
    sh.set_kernel(*DIRECT)
    sh.step(n)
    return end(W, sh)


@pytest.mark.parametrize("storage,tile", [("f32", (1, 8)), ("f32", (2, 16)), ("bf16", (0, 8)), ("bf16sr", (1, 16))])
def test_graph_replays_across_runs(W, storage, tile):
    """Four runs of ten steps with a set tile, two replays of one captured graph each,
    host reads in between: the members keep their order, so the graph of the first run
    is replayed against the tables of the later ones."""
    say(f"case graph replays {storage} {tile}")
    b = W.Batch(storage=storage.replace("sr", ""), max_shots=4)
    b.set_kernel(*tile)
    b.set_graph(5)
    shots = [make(W, *g, storage, seed=i) for i, g in enumerate(SMALL)]
    for sh in shots:
        b.add(sh, 40)
    for run in range(1, 5):
        b.run(10)
        for i, sh in enumerate(shots):
            same(end(W, sh, close=False), solo_steps(W, i, storage, 10 * run), (run, i))
    b.close()
    for sh in shots:
        sh.close()


@pytest.mark.parametrize("graph", [0, 2])
@pytest.mark.parametrize("tile", [(4, 4), (1, 8), (0, 16)])
def test_membership_and_streams(W, tile, graph):
    """A member that joins midway, one that leaves and continues on its own, members set
    up on a stream other than the batch's."""
    import torch
    say(f"case membership {tile} graph {graph}")
    side = torch.cuda.Stream()
    b = W.Batch(max_shots=4)
    b.set_kernel(*tile)
    b.set_graph(graph)
    m = [make(W, *g, "f32", seed=i, stream=side if i % 2 else None) for i, g in enumerate(SMALL)]
    total = [23, 30, 17, 26]
    b.add(m[0], total[0])
    b.add(m[1], total[1])
    b.run(5)
    b.add(m[2], total[2])
    b.run(3)
    b.remove(m[1])
    m[1].step(total[1] - 8)
    b.add(m[3], total[3])
    b.run(100)
    for i, sh in enumerate(m):
        same(end(W, sh), solo_steps(W, i, "f32", total[i]), (tile, i))
    b.close()


@pytest.mark.parametrize("storage,grids", [("bf16", [(395, 352, 331, 20, False), (163, 585, 570, 20, False),
                                                     (300, 300, 300, 20, True)]),
                                           ("f16", [(384, 360, 331, 20, False)]), ("f32", [(300, 300, 290, 20, False)])])
def test_batch_of_streaming_members(W, storage, grids):
    """Members past the block kernel's sizes without a set tile: two points per lane,
    one where 128-wide tiles leave a third of the lanes idle, one with an eta array,
    beside small ones, in captured steps and plain ones."""
    say(f"case batch of streaming members {storage}")
    specs = [(g[:4], g[4]) for g in grids] + [((60, 44, 30, 4), False), ((70, 30, 30, 4), True)]
    n = [3, 5, 4, 5, 2]
    b = W.Batch(storage=storage, max_shots=len(specs))
    b.set_graph(2)
    shots = [make(W, *g, storage, True, eta, 2, seed=i) for i, (g, eta) in enumerate(specs)]
    for sh, k in zip(shots, n):
        b.add(sh, k)
    b.run(3)
    b.run(2)
    b.close()
    for i, (g, eta) in enumerate(specs):
        solo = make(W, *g, storage, True, eta, 2, seed=i)
        solo.set_kernel(*DIRECT)
        solo.step(n[i])
        same(end(W, shots[i]), end(W, solo), (storage, i))


def test_small_members_of_every_kind(W):
    """Small members with damping off share launches with those that have a layer: a
    layer width that the flag switches off among them."""
    say("case small members of every kind")
    specs = [(70, 45, 37, 5, True, False, 1), (64, 40, 36, 0, False, False, 2), (33, 50, 41, 8, False, False, 1),
             (90, 30, 30, 6, True, True, 1), (50, 50, 50, 9, True, False, 6), (48, 33, 20, 0, False, False, 7)]
    for pieces in ((1, 1, 2, 4, 9), (12,)):
        n = [5, 9, 12, 7, 10, 3]
        b = W.Batch(max_shots=8)
        shots = [make(W, *m[:4], "f32", m[4], m[5], m[6], seed=i) for i, m in enumerate(specs)]
        for sh, k in zip(shots, n):
            b.add(sh, k)
        for k in pieces:
            b.run(k)
        b.close()
        for i, m in enumerate(specs):
            solo = make(W, *m[:4], "f32", m[4], m[5], m[6], seed=i)
            solo.set_kernel(*DIRECT)
            solo.step(n[i])
            same(end(W, shots[i]), end(W, solo), (pieces, i))
