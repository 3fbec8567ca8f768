"""A voxel that is not finite reaches the voxels whose sums take it, and no
others, under any split: R per Gaussian stage, in one iteration 2 R with the RSF
force (K*(H I), then K*g) and R with the Sec. 4.2 force."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf as mod
    return mod


def evolve(rsf, I, phi0, radius, force, storage, iters, waves=0):
    import torch
    f = rsf.RSF_FORCE_PAPER if force == "paper" else rsf.RSF_FORCE_RSF
    p = rsf.make_params(radius / 3 - 0.05, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage, force=f)
    with rsf.Context(0) as ctx:
        ctx.set_split_targets(waves, 0, 0)
        phi = torch.from_numpy(phi0).cuda()
        ctx.evolve_ex(torch.from_numpy(I).cuda(), phi, p, iters)
        torch.cuda.synchronize()
    return phi.cpu().numpy()


def fields(shape):
    rng = np.random.Generator(np.random.PCG64(29))
    return (rng.uniform(0.0, 1.0, shape).astype(np.float32),
            rng.uniform(-3.0, 3.0, shape).astype(np.float32))


# (nz, ny, nx) and the voxel: the small-volume form of the xy pass (one and two
# strips), the march with 4 and with 8 waves, several strips and row chunks; near
# a face, at rows and columns of every remainder of four
SHAPES = [((9, 50, 60), (4, 21, 30)), ((5, 47, 140), (2, 0, 63)), ((70, 130, 90), (35, 66, 45)),
          ((3, 90, 300), (1, 43, 131)), ((40, 64, 512), (20, 31, 257)), ((3, 33, 760), (1, 16, 254))]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("radius,storage", [(1, "f32"), (4, "f16"), (6, "f32"), (9, "f32"), (9, "bf16"),
                                            (11, "f16"), (14, "f32")])
@pytest.mark.parametrize("force", ["rsf", "paper"])
@pytest.mark.parametrize("shape,at", SHAPES)
def test_one_iteration_reaches_the_window_only(rsf, shape, at, force, radius, storage, value):
    I, phi0 = fields(shape)
    clean = evolve(rsf, I, phi0, radius, force, storage, 1)
    I[at] = value
    got = evolve(rsf, I, phi0, radius, force, storage, 1)
    reach = radius if force == "paper" else 2 * radius
    box = np.zeros(shape, bool)
    box[tuple(slice(max(a - reach, 0), a + reach + 1) for a in at)] = True
    assert np.array_equal(~np.isfinite(got), box)
    assert np.array_equal(got[~box], clean[~box])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(64, 64, 64), (20, 71, 150), (3, 90, 520)])
def test_any_split_gives_the_same_phi(rsf, shape, storage):
    """Voxels that are not finite, and (FP16) g that overflows, in three
    iterations: the small form and the march in any row chunks."""
    I, phi0 = fields(shape)
    I[1, 33, 20], I[2, 50, 41] = float("nan"), float("-inf")
    I[0, 5:9, 50:60] = 400.0
    out = [evolve(rsf, I, phi0, 4, "rsf", storage, 3, w) for w in (0, 16, 1 << 20)]
    assert np.isfinite(out[0]).any() and not np.isfinite(out[0]).all()
    for o in out[1:]:
        assert np.array_equal(o, out[0], equal_nan=True)


def test_a_tile_in_a_batch_is_the_tile_alone(rsf):
    import torch
    p = rsf.make_params(2.95, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0)
    vols, phis, alone = [], [], []
    for k, shape in enumerate([(20, 64, 400), (24, 70, 512), (16, 50, 130)]):
        I, phi0 = fields(shape)
        I[3, 20 + k, 61 + k] = float("nan")
        vols.append(torch.from_numpy(I).cuda())
        phis.append(torch.from_numpy(phi0).cuda())
        alone.append(evolve(rsf, I, phi0, 9, "rsf", "f32", 2))
    with rsf.Context(0) as ctx:
        ctx.evolve_batch(vols, phis, p, 2)
        torch.cuda.synchronize()
    for phi, a in zip(phis, alone):
        assert np.array_equal(phi.cpu().numpy(), a, equal_nan=True)
