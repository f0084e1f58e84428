"""Two steps per launch in 3D over the lengths of z-chunk that its plan takes:
one plane, fewer planes than the shortest chunk, a short last chunk, and plane
counts around 32, bitwise against one step per launch."""
import numpy as np
import pytest

from paper_2108_08591_amd import cases as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("sets", ["all", "velocity"])
@pytest.mark.parametrize("dims,walls", [((40, 12, 1), False), ((33, 9, 3), True), ((31, 70, 5), False),
                                        ((96, 96, 33), True), ((138, 148, 61), False), ((65, 130, 95), True)])
def test_chunks(storage, sets, dims, walls):
    from paper_2108_08591_amd import mdf
    bc = [C.WALL if walls else C.PERIODIC] * 6
    wall = np.zeros((6, 3))
    if walls:
        wall[3, 0] = 0.05
    spec = C.CaseSpec(C.D3Q7, dims, C.s1_for_nu(0.05, C.D3Q7), bc=tuple(bc), wall_u=wall)
    spec.s2 = 1.2
    gen = torch.Generator().manual_seed(sum(dims))
    data = (0.02 * torch.randn((4,) + spec.fshape, generator=gen, dtype=torch.float64)).to("cuda:0")
    data = data.to(torch.float64 if storage == "f64" else torch.float32)
    out = []
    for form in (0, 2):
        s = mdf.Solver(spec, storage=storage, init=("fields", [data]), u_ref=0.1, sets=sets)
        s.set_launch(64, 4, 8, form)
        s.step(7)
        out.append(torch.as_tensor(s.moments(0)).clone())
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
