"""Launches of several steps in 2D (tiles, small and large, and strips of
columns) against one-step launches of the same context.

The two give the same bits: every population, every field emitted at the end
of a call and every sum of accumulated fields, whatever the remainder of the
grid in tiles or strips, at walls, across periodic faces, around obstacles
and with a force field under Scheme II.  One-step launches are checked
against the oracle elsewhere."""
import numpy as np
import pytest
import torch

from paper_2108_08591_amd import cases as C
from paper_2108_08591_amd import mdf

pytestmark = pytest.mark.gpu

ALL = mdf.FIELD_ALL


def _spec(nx, ny, wallx, wally, rng, lattice=C.D2Q5, scheme2=False):
    bc, wall = [C.PERIODIC] * 6, np.zeros((6, 3))
    for axis, on in ((0, wallx), (1, wally)):
        if on:
            bc[2 * axis] = bc[2 * axis + 1] = C.WALL
            wall[2 * axis:2 * axis + 2, :2] = rng.uniform(-0.1, 0.1, (2, 2))
    spec = C.CaseSpec(lattice, (nx, ny), 1.1, bc=tuple(bc), wall_u=wall, force=(1e-4, -2e-4, 0.0))
    if scheme2:
        spec.forcing = 1
    return spec


def _outputs(spec, storage, form, steps, fields, mask, force, sets="all"):
    data = fields.to(torch.float64 if storage == "f64" else torch.float32)
    s = mdf.Solver(spec, storage=storage, solid=None if mask is None else [mask], init=("fields", [data]), u_ref=0.1,
                   sets=sets)
    s.set_launch(64, 4, 8, form)
    if force is not None:
        s.set_force_field(force)
    s.step(steps)
    out = [s.populations()]
    acc = [torch.zeros_like(t) for t in s.new_field_buffers(ALL)]
    s.step_emit(steps, ALL | mdf.FIELD_ACCUMULATE, acc)
    out += acc
    out += s.step_emit(steps + 1, ALL)
    out.append(s.gradients(ALL))
    return out


def _compare(spec, storage, steps, mask=None, force=None, sets="all", label=""):
    nx, ny = spec.shape
    g = torch.Generator().manual_seed(nx * 7919 + ny)
    fields = (torch.rand(3, ny, nx, generator=g, dtype=torch.float64) - 0.5) * 0.1
    if mask is not None:
        fields[:, torch.as_tensor(mask).bool()] = 0.0
    print(f"[gpu] several steps {label} {nx}x{ny} {storage} steps {steps}", flush=True)
    one = _outputs(spec, storage, 0, steps, fields, mask, force, sets)
    many = _outputs(spec, storage, 2, steps, fields, mask, force, sets)
    for k, (a, b) in enumerate(zip(one, many)):
        assert torch.isfinite(a).all(), f"{label}: output {k} not finite"
        assert torch.equal(a, b), f"{label}: output {k} differs by {(a - b).abs().max().item():.3e}"


# remainders of the tiles (8, 24 columns; 8, 24 rows) and sizes below them;
# 288 x 256 and 289 x 257 lie on either side of the change of tile
TILE_SIZES = [(1, 1), (2, 9), (8, 8), (9, 7), (24, 25), (33, 17), (64, 64), (224, 219), (300, 170), (288, 256),
              (289, 257), (25, 3001), (3001, 25)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev", "bf16dev"])
@pytest.mark.parametrize("wallx,wally", [(False, False), (True, False), (False, True), (True, True)])
def test_tiles_equal_one_step_launches(storage, wallx, wally):
    for n, (nx, ny) in enumerate(TILE_SIZES):
        rng = np.random.default_rng(n)
        mask = (rng.random((ny, nx)) < 0.1).astype(np.uint8) if n % 2 and nx > 2 else None
        _compare(_spec(nx, ny, wallx, wally, rng), storage, (4, 5, 8, 12)[n % 4], mask, label="tiles")


@pytest.mark.parametrize("storage,nx,ny", [("f32", 1537, 1473), ("f32", 49, 46000), ("f32", 64, 36000),
                                           ("f16dev", 2073, 2200), ("bf16dev", 57, 79001)])
def test_strips_equal_one_step_launches(storage, nx, ny):
    """Beyond the Infinity Cache: strips of 48 (FP32) and 56 columns, ragged
    and narrower than one strip, chunks with a remainder."""
    rng = np.random.default_rng(nx)
    for k, (wallx, wally) in enumerate([(True, True), (False, False), (True, False)]):
        mask = (rng.random((ny, nx)) < 0.02).astype(np.uint8) if k != 1 else None
        _compare(_spec(nx, ny, wallx, wally, rng), storage, (5, 7, 9)[k], mask, label="strips")


@pytest.mark.parametrize("storage,nx,ny", [("f64", 70, 45), ("f32", 70, 45), ("f32", 1500, 1520), ("f16dev", 2100, 2201)])
def test_force_field_and_scheme2(storage, nx, ny):
    rng = np.random.default_rng(5)
    mask = (rng.random((ny, nx)) < 0.05).astype(np.uint8)
    force = torch.as_tensor(rng.uniform(-1e-4, 1e-4, (2, ny, nx)))
    for scheme2 in (False, True):
        _compare(_spec(nx, ny, True, False, rng, scheme2=scheme2), storage, 5, mask, force, label="forced")


@pytest.mark.parametrize("lattice,sets", [(C.D2Q5, "velocity"), (mdf.D2Q4, "all"), (mdf.D2Q4, "velocity")])
def test_other_lattices(lattice, sets):
    for storage, nx, ny in (("f64", 90, 41), ("f32", 90, 41), ("f32", 1700, 2300)):
        rng = np.random.default_rng(nx)
        _compare(_spec(nx, ny, True, True, rng, lattice), storage, 8, sets=sets, label="lattice")


@pytest.mark.parametrize("storage,sizes", [("f64", [(64, 64)] * 3), ("f64", [(200, 130), (64, 64), (33, 300), (128, 128)]),
                                           ("f32", [(1200, 1100), (64, 64), (1000, 1001)])])
def test_batches_with_cases_switched_off(storage, sizes):
    """A batch whose active set shrinks and grows between chunks of the same
    length (replayed graphs), in small tiles, large tiles and strips."""
    stream = torch.cuda.Stream()
    outs = []
    for form in (0, 2):
        rng = np.random.default_rng(3)
        specs = [_spec(nx, ny, k % 2 == 0, True, rng) for k, (nx, ny) in enumerate(sizes)]
        print(f"[gpu] several steps batch {storage} form {form}", flush=True)
        with torch.cuda.stream(stream):
            s = mdf.Solver(specs, storage=storage, stream=stream)
            s.set_launch(64, 4, 8, form)
            s.step(9)
            s.set_active([k != 1 for k in range(len(sizes))])
            s.step(9)
            s.set_active([1] * len(sizes))
            for _ in range(3):
                s.step(9)
            res = s.run_steady(1e-15, 7, 21)
            outs.append([s.populations(k) for k in range(len(sizes))] + [torch.as_tensor(res[1])])
        stream.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a, b)
