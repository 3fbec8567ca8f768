"""Every form of the iteration's xy pass against another one, bitwise: a step of
evolve (the form its plan takes, which the plan's own test asserts) against the
one-step probe, which marches with workgroups of 4 waves, and a tile of a batch
against the tile alone."""
import numpy as np
import pytest

from xy_forms import BATCHES, VOLUMES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf as mod
    return mod


def fields(shape, seed):
    import torch
    rng = np.random.Generator(np.random.PCG64(seed))
    return (torch.from_numpy(rng.random(shape, dtype=np.float32)).cuda(),
            torch.from_numpy(rng.random(shape, dtype=np.float32) * 6 - 3).cuda())


def params(rsf, radius, storage):
    return rsf.make_params(radius / 3 - 0.05, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("radius,shape,waves,chunks", VOLUMES)
def test_a_step_is_the_probe(rsf, radius, shape, waves, chunks, storage):
    import torch
    if storage != "f32" and not 4 <= radius <= 12:
        pytest.skip("16-bit fields are built for radii 4 to 12")
    vol, phi = fields(shape, 41)
    p = params(rsf, radius, storage)
    with rsf.Context(0) as ctx:
        want = ctx.probe(vol, phi, p)["phi_next"]
        ctx.evolve_ex(vol, phi, p, 1)
        torch.cuda.synchronize()
    assert torch.equal(phi, want)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("radius,shapes,waves", BATCHES)
def test_a_tile_of_a_batch_is_the_tile_alone(rsf, radius, shapes, waves, storage):
    import torch
    p = params(rsf, radius, storage)
    vols, phis = zip(*[fields(s, 43 + k) for k, s in enumerate(shapes)])
    with rsf.Context(0) as ctx:
        alone = [phi.clone() for phi in phis]
        for vol, phi in zip(vols, alone):
            ctx.evolve_ex(vol, phi, p, 3)
        ctx.evolve_batch(list(vols), list(phis), p, 3)
        torch.cuda.synchronize()
    for phi, want in zip(phis, alone):
        assert torch.equal(phi, want)
