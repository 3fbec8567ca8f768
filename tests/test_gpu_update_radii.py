"""The fused update against the separate passes, bitwise, at the radii where
its form changes: taps in vector or in scalar registers, 32-bit or 64-bit slice
addresses, packed or FP32 rings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# sigma -> radius ceil(3 sigma): 6, 7, 8, 9 (FP32 rings, the form changes after
# 7), 10, 11, 12 (packed ring, after 10)
CASES = [("f32", "f32", 2.0), ("f32", "f32", 2.3), ("f32", "f32", 2.6), ("f32", "f32", 3.0),
         ("u16", "f32", 2.3), ("u16", "f32", 2.6), ("u16", "bf16", 2.3), ("u16", "bf16", 2.6),
         ("f32", "f16", 3.3), ("u16", "f16", 3.3), ("u16", "f16", 3.6), ("u16", "f16", 4.0)]


@pytest.mark.parametrize("image,storage,sigma", CASES)
def test_fused_update_is_the_separate_passes(image, storage, sigma):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf
    # two blocks of up to 27 unrolled steps, the rest step by step; a tile
    # column and row more than one workgroup's
    shape = (75, 9, 67)
    rng = np.random.Generator(np.random.PCG64(17))
    I = rng.uniform(0.0, 1.0, shape).astype(np.float32)
    if image == "u16":
        I = np.round(I * 65535.0).astype(np.uint16)
    phi0 = torch.from_numpy(rng.uniform(-3.0, 3.0, shape).astype(np.float32)).cuda()
    vol = torch.from_numpy(I).cuda()
    p = rsf.make_params(sigma, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage)
    out = []
    with rsf.Context(0) as ctx:
        ctx.set_split_targets(0, 0, 1)   # the update whole in z, which lets it fuse
        for fuse in (False, True):
            ctx.set_fusion(fuse)
            phi = phi0.clone()
            ctx.profile(True)
            ctx.evolve_ex(vol, phi, p, 4)
            torch.cuda.synchronize()
            ctx.profile(False)
            out.append((phi, ctx.profile_read()["z_heaviside"][0]))
    assert torch.equal(out[0][0], out[1][0])
    assert (out[0][1], out[1][1]) == (4, 1)


# chunks of 2 to 4 slices in the update pass and of 2 to 8 in the z pass, with a
# shorter last one
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(9, 9, 9), (13, 20, 30), (64, 64, 64), (45, 71, 67), (31, 8, 64)])
def test_short_z_chunks_do_not_change_phi(shape, storage):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf
    rng = np.random.Generator(np.random.PCG64(19))
    vol = torch.from_numpy(rng.uniform(0.0, 1.0, shape).astype(np.float32)).cuda()
    phi0 = torch.from_numpy(rng.uniform(-3.0, 3.0, shape).astype(np.float32)).cuda()
    p = rsf.make_params(3.0, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage)
    out = []
    with rsf.Context(0) as ctx:
        ctx.set_fusion(False)
        for z, u in ((0, 0), (1, 1)):   # its own chunks; whole in z
            ctx.set_split_targets(0, z, u)
            phi = phi0.clone()
            ctx.evolve_ex(vol, phi, p, 3)
            torch.cuda.synchronize()
            out.append((phi, ctx.stats(cap=0)[2]))
    assert torch.equal(out[0][0], out[1][0])
    # FP64 sums of the same terms in another order
    assert out[0][1] == pytest.approx(out[1][1], rel=1e-12)
