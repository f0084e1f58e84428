"""The kernels of launches of several steps in 2D that a call picks by its
options, bitwise against one-step launches (which are checked against the
oracle elsewhere)."""
import numpy as np
import pytest
import torch

from paper_2108_08591_amd import cases as C, mdf
from test_gpu_several_steps import _compare, _spec

pytestmark = pytest.mark.gpu

MOM = mdf.FIELD_MOMENTS
# a remainder of the tiles, small and large, and strips (FP32 and 16-bit beyond
# the Infinity Cache)
GRIDS = [("f64", 70, 45), ("f64", 300, 259), ("f32", 300, 259), ("f32", 1500, 1520), ("f16dev", 300, 259),
         ("f16dev", 2100, 2201), ("bf16dev", 2100, 2201)]


def _init(nx, ny, storage, seed=0):
    g = torch.Generator().manual_seed(seed + nx)
    data = (torch.rand(3, ny, nx, generator=g, dtype=torch.float64) - 0.5) * 0.1
    return data.to(torch.float64 if storage == "f64" else torch.float32)


@pytest.mark.parametrize("storage,nx,ny", GRIDS)
@pytest.mark.parametrize("scheme2", [False, True])
@pytest.mark.parametrize("mask", [False, True])
def test_forced_without_and_with_emission(storage, nx, ny, scheme2, mask):
    """Force field and Scheme II, with a mask and without: steps alone (a kernel
    of its own each), then steps that emit (one kernel for both)."""
    print(f"[gpu] forced {storage} {nx}x{ny} scheme2={scheme2} mask={mask}", flush=True)
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(nx)
        data = _init(nx, ny, storage)
        solid = (rng.random((ny, nx)) < 0.05).astype(np.uint8) if mask else None
        if mask:
            data[:, torch.as_tensor(solid).bool()] = 0.0
        s = mdf.Solver(_spec(nx, ny, True, False, rng, scheme2=scheme2), storage=storage,
                       solid=[solid] if mask else None, init=("fields", [data]), u_ref=0.1)
        s.set_launch(64, 4, 8, form)
        if not scheme2:
            s.set_force_field(torch.as_tensor(rng.uniform(-1e-4, 1e-4, (2, ny, nx))))
        s.step(8)
        got = [s.populations()]
        s.step(4)
        out.append(got + [s.populations()] + s.step_emit(9, MOM))
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,sizes", [("f64", [(70, 45), (33, 90)]), ("f32", [(1200, 1100), (64, 64)]),
                                           ("f16dev", [(2100, 1600), (57, 300)])])
def test_forced_batches(storage, sizes):
    """A batch in which one case has a force field and no case a mask."""
    print(f"[gpu] forced batch {storage} {sizes}", flush=True)
    stream = torch.cuda.Stream()
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(7)
        specs = [_spec(nx, ny, True, k % 2 == 0, rng) for k, (nx, ny) in enumerate(sizes)]
        init = [_init(nx, ny, storage, k) for k, (nx, ny) in enumerate(sizes)]
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, init=("fields", init), u_ref=0.1, stream=stream)
            s.set_launch(64, 4, 8, form)
            nx, ny = sizes[1]
            s.set_force_field(torch.as_tensor(rng.uniform(-1e-4, 1e-4, (2, ny, nx))), case=1)
            for _ in range(3):
                s.step(8)
            out.append([s.populations(k) for k in range(2)] + s.step_emit(9, MOM))
        stream.synchronize()
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,nx,ny", GRIDS)
@pytest.mark.parametrize("mask", [False, True])
def test_calls_of_three_steps(storage, nx, ny, mask):
    """Three steps a call, two of them in one launch: plain, accumulating (both
    steps count) and emitting, and a force field."""
    print(f"[gpu] three steps {storage} {nx}x{ny} mask={mask}", flush=True)
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(nx)
        data = _init(nx, ny, storage)
        solid = (rng.random((ny, nx)) < 0.05).astype(np.uint8) if mask else None
        if mask:
            data[:, torch.as_tensor(solid).bool()] = 0.0
        s = mdf.Solver(_spec(nx, ny, mask, True, rng), storage=storage, solid=[solid] if mask else None,
                       init=("fields", [data]), u_ref=0.1)
        s.set_launch(64, 4, 8, form)
        s.step(3)
        got = [s.populations()]
        acc = [torch.zeros_like(t) for t in s.new_field_buffers(MOM)]
        s.step_emit(3, MOM | mdf.FIELD_ACCUMULATE, acc)
        got += acc + s.step_emit(3, MOM)
        s.set_force_field(torch.as_tensor(rng.uniform(-1e-4, 1e-4, (2, ny, nx))))
        s.step(3)
        out.append(got + [s.gradients(mdf.FIELD_ALL)])
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,sizes", [("f64", [(70, 45), (33, 90), (1, 7)]), ("f32", [(1200, 1100), (64, 64)])])
@pytest.mark.parametrize("mask", [False, True])
def test_batches_of_three_steps(storage, sizes, mask):
    """Batched two-step launches, in chunks of three and six steps, while cases
    are switched off and on."""
    print(f"[gpu] three steps batch {storage} {sizes} mask={mask}", flush=True)
    stream = torch.cuda.Stream()
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(7)
        specs = [_spec(nx, ny, True, k % 2 == 0, rng) for k, (nx, ny) in enumerate(sizes)]
        init = [_init(nx, ny, storage, k) for k, (nx, ny) in enumerate(sizes)]
        solid = None
        if mask:
            solid = [(rng.random((ny, nx)) < 0.05).astype(np.uint8) if k == 0 else None
                     for k, (nx, ny) in enumerate(sizes)]
            init[0][:, torch.as_tensor(solid[0]).bool()] = 0.0
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, solid=solid, init=("fields", init), u_ref=0.1, stream=stream)
            s.set_launch(64, 4, 8, form)
            s.step(3)
            s.set_active([k != 1 for k in range(len(sizes))])
            s.step(6)
            s.set_active([1] * len(sizes))
            for _ in range(3):
                s.step(6)
            res = s.run_steady(1e-15, 3, 9)
            out.append([s.populations(k) for k in range(len(sizes))] + [torch.as_tensor(res[1])] + s.step_emit(3, MOM))
        stream.synchronize()
    assert all(torch.isfinite(t.double()).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,sizes", [("f32", [(1200, 1100), (64, 64), (1000, 1001), (300, 290)]),
                                           ("f16dev", [(57, 61), (1700, 1600), (500, 410), (1500, 1300)])])
def test_units_follow_the_running_cases(storage, sizes):
    """A batch beyond the Infinity Cache whose running cases go from all of them
    (strips) to a middle one (large tiles) and a small one (small tiles) and
    back, each set twice with chunks of one length, so that captured launches
    of several grids are replayed."""
    print(f"[gpu] units of running cases {storage}", flush=True)
    sets = [[1, 1, 1, 1], [0, 0, 0, 1], [1, 1, 1, 1], [0, 1, 0, 0], [1, 0, 0, 0], [0, 0, 1, 1], [1, 0, 0, 0],
            [0, 1, 0, 0], [0, 0, 0, 1], [1, 1, 1, 1]]
    stream = torch.cuda.Stream()
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(11)
        specs = [_spec(nx, ny, k % 2 == 0, True, rng) for k, (nx, ny) in enumerate(sizes)]
        init = [_init(nx, ny, storage, k) for k, (nx, ny) in enumerate(sizes)]
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, init=("fields", init), u_ref=0.1, stream=stream)
            s.set_launch(64, 4, 8, form)
            for active in sets:
                s.set_active(active)
                s.step(9)
                s.step(9)
            s.set_active([1] * 4)
            out.append([s.populations(k) for k in range(4)] + s.step_emit(9, MOM))
            stats = s.graph_stats()
        stream.synchronize()
        assert stats["failed"] == 0 and stats["replayed"] == 2 * len(sets) + 1
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,sizes", [("f32", [(1200, 1100), (64, 64), (1000, 1001)]),
                                           ("f16dev", [(1700, 1600), (57, 300), (1500, 1300)])])
def test_accumulation_beyond_the_cache_in_batches(storage, sizes):
    """Accumulated fields (tiles) between steps and emission (strips) of a batch
    beyond the Infinity Cache, in chunks of one length."""
    print(f"[gpu] accumulation batch {storage}", flush=True)
    stream = torch.cuda.Stream()
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(13)
        specs = [_spec(nx, ny, k % 2 == 0, True, rng) for k, (nx, ny) in enumerate(sizes)]
        init = [_init(nx, ny, storage, k) for k, (nx, ny) in enumerate(sizes)]
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, init=("fields", init), u_ref=0.1, stream=stream)
            s.set_launch(64, 4, 8, form)
            acc = [torch.zeros_like(t) for t in s.new_field_buffers(MOM)]
            s.step(9)
            s.step_emit(9, MOM | mdf.FIELD_ACCUMULATE, acc)
            s.step(9)
            s.step_emit(9, MOM | mdf.FIELD_ACCUMULATE, acc)
            out.append(acc + s.step_emit(9, MOM) + [s.populations(k) for k in range(3)])
        stream.synchronize()
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,nx,ny,longest", [("f64", 70, 45, 4), ("f64", 300, 259, 4), ("f32", 70, 45, 4),
                                                   ("f32", 300, 259, 4), ("f32", 1500, 1520, 5), ("f16dev", 70, 45, 4),
                                                   ("f16dev", 300, 259, 4), ("f16dev", 2100, 2201, 4),
                                                   ("bf16dev", 2100, 2201, 4)])
@pytest.mark.parametrize("mask", [False, True])
@pytest.mark.parametrize("walls", [False, True])
def test_every_length_of_launch(storage, nx, ny, longest, mask, walls):
    """Calls of K + 1 steps, one launch of K and one of one (five only without a
    mask: with one, three and two), plain, emitting and accumulating."""
    print(f"[gpu] every length {storage} {nx}x{ny} mask={mask} walls={walls}", flush=True)
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(nx)
        data = _init(nx, ny, storage)
        solid = (rng.random((ny, nx)) < 0.05).astype(np.uint8) if mask else None
        if mask:
            data[:, torch.as_tensor(solid).bool()] = 0.0
        s = mdf.Solver(_spec(nx, ny, walls, walls, rng), storage=storage, solid=[solid] if mask else None,
                       init=("fields", [data]), u_ref=0.1)
        s.set_launch(64, 4, 8, form)
        got = []
        for k in range(2, longest + 1):
            s.step(k + 1)
            got += [s.moments()] + s.step_emit(k + 1, MOM)
            acc = [torch.zeros_like(t) for t in s.new_field_buffers(MOM)]
            s.step_emit(k + 1, MOM | mdf.FIELD_ACCUMULATE, acc)
            got += acc
        out.append(got + [s.populations()])
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage,sizes,n", [("f32", [(1200, 1100), (64, 64), (1000, 1001)], 6),
                                             ("f32", [(1200, 1100), (64, 64), (1000, 1001)], 11),
                                             ("f16dev", [(1700, 1600), (57, 300), (1500, 1300)], 5)])
@pytest.mark.parametrize("mask", [False, True])
def test_longest_launches_in_batches(storage, sizes, n, mask):
    """Strips of a batch at their longest launch, plain and emitting."""
    print(f"[gpu] longest launches batch {storage} n={n} mask={mask}", flush=True)
    stream = torch.cuda.Stream()
    out = []
    for form in (0, 2):
        rng = np.random.default_rng(17)
        specs = [_spec(nx, ny, k % 2 == 0, True, rng) for k, (nx, ny) in enumerate(sizes)]
        init = [_init(nx, ny, storage, k) for k, (nx, ny) in enumerate(sizes)]
        solid = None
        if mask:
            solid = [(rng.random((ny, nx)) < 0.05).astype(np.uint8) if k != 1 else None
                     for k, (nx, ny) in enumerate(sizes)]
            for t, m in zip(init, solid):
                if m is not None:
                    t[:, torch.as_tensor(m).bool()] = 0.0
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, solid=solid, init=("fields", init), u_ref=0.1, stream=stream)
            s.set_launch(64, 4, 8, form)
            s.step(n)
            out.append([s.populations(k) for k in range(3)] + s.step_emit(n, MOM) + [s.populations(0)])
        stream.synchronize()
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("storage", ["f16dev", "bf16dev"])
def test_two_steps_on_large_periodic_grids(storage):
    """Periodic grids of more than 3.5 million nodes inside the Infinity Cache:
    two steps per launch, then, between steps that emit, tiles."""
    nx, ny = 2003, 1801
    print(f"[gpu] large periodic {storage} {nx}x{ny}", flush=True)
    out = []
    for form in (0, 2):
        s = mdf.Solver(_spec(nx, ny, False, False, None), storage=storage, init=("fields", [_init(nx, ny, storage)]),
                       u_ref=0.1)
        s.set_launch(64, 4, 8, form)
        s.step(4)
        got = [s.populations()]
        s.step(9)
        got += [s.populations()] + s.step_emit(6, MOM)
        s.step(6)
        out.append(got + [s.populations()])
    assert all(torch.isfinite(t).all() for t in out[0])
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("lattice", [C.D2Q5, mdf.D2Q4])
@pytest.mark.parametrize("mask", [False, True])
@pytest.mark.parametrize("steps", [3, 8, 9])
def test_two_steps_that_accumulate_many_channels(lattice, mask, steps):
    """FP64, all channels accumulated by two sets and, on a small grid, by three:
    two steps per launch, after and before launches of up to four."""
    for nx, ny, sets in ((300, 259, "velocity"), (391, 401, "all")):
        rng = np.random.default_rng(5)
        solid = (rng.random((ny, nx)) < 0.1).astype(np.uint8) if mask else None
        _compare(_spec(nx, ny, mask, False, rng, lattice), "f64", steps, solid, sets=sets, label=sets)
