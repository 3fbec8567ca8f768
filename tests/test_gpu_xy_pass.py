"""The iteration's xy pass at the sizes where its strips, row groups and chunks
can go wrong, against the FP64 oracle.

A workgroup covers up to 256 or 512 columns (64 per wave) and marches a chunk
of rows four at a time; neighbouring strips share R columns with the RSF force
and the last strip is moved left to its full width."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf as mod
    return mod


def fields(shape, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    I = rng.uniform(0.0, 1.0, shape).astype(np.float32)
    phi = rng.uniform(-3.0, 3.0, shape).astype(np.float32)
    return I, phi


# (nz, ny, nx): one wave, a wave's edge, one strip of 4 and of 8 waves and one
# column more, several strips with a ragged last one; rows fewer than a group,
# than the radius, and off every multiple of four
SHAPES = [(3, 3, 63), (3, 5, 64), (3, 30, 65), (4, 37, 256), (3, 41, 257), (3, 18, 300),
          (3, 7, 512), (3, 22, 513), (3, 19, 705), (3, 133, 5)]


@pytest.mark.parametrize("sigma", [0.3, 1.3, 3.0, 3.4, 4.9, 5.3])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("force", ["rsf", "paper"])
def test_one_iteration_matches_the_oracle(rsf, shape, sigma, force):
    import torch
    I, phi0 = fields(shape, 7)
    f = rsf.RSF_FORCE_PAPER if force == "paper" else rsf.RSF_FORCE_RSF
    coef = dict(sigma=sigma, lambda1=1.0, lambda2=1.5, nu=0.001, mu=1.0, dt=0.1, eps=1.0)
    p = rsf.make_params(force=f, **coef)
    with rsf.Context(0) as ctx:
        vol, phi = torch.from_numpy(I).cuda(), torch.from_numpy(phi0).cuda()
        ctx.evolve_ex(vol, phi, p, 1)
        torch.cuda.synchronize()
        got = phi.cpu().numpy().astype(np.float64)
    want, _ = oracle.evolve(I, phi0, oracle.params_array(eta=1e-10, force=1 if force == "paper"
                                                         else 0, **coef), 1)
    # one step moves phi by dt E, and E's terms are differences of O(1) to
    # O(10) fields whose FP32 values are within 2e-5 (the probe bar): 0.1 * 2e-5
    # on top of phi's own rounding (3 * 2^-24)
    assert float(np.max(np.abs(got - want))) <= 2.5e-6


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(5, 150, 70), (3, 90, 520)])
def test_row_chunks_do_not_change_phi(rsf, shape, storage):
    """Any number of row chunks gives bitwise the same phi: each output row's
    sums are taken over the same rows in the same order."""
    import torch
    I, phi0 = fields(shape, 11)
    p = rsf.make_params(3.0, 1.0, 1.0, 0.001, 1.0, 0.1, 1.0, storage=storage)
    out = []
    with rsf.Context(0) as ctx:
        vol = torch.from_numpy(I).cuda()
        for waves in (0, 16, 4096, 1 << 20):
            ctx.set_split_targets(waves, 0, 0)
            phi = torch.from_numpy(phi0).cuda()
            ctx.evolve_ex(vol, phi, p, 3)
            torch.cuda.synchronize()
            out.append(phi)
    for o in out[1:]:
        assert torch.equal(o, out[0])


# LDS of the small-volume form from 43 KB (sigma 1.3, one wave of columns) to
# 146 KB; one, two and three strips of 128 columns, a last strip of its own
# width, chunks of 2 to 16 rows, rows off every multiple of four
SMALL = [((64, 64, 64), 3.0), ((45, 71, 67), 3.0), ((3, 30, 65), 2.9), ((5, 18, 127), 1.3),
         ((7, 33, 150), 3.0), ((40, 64, 100), 3.9), ((30, 41, 257), 1.6), ((64, 63, 64), 5.3)]


TYPES = [("f32", "f32"), ("u16", "f16"), ("u16", "f32"), ("f32", "bf16")]


# (mixed types are built for radii of up to 12)
@pytest.mark.parametrize("shape,sigma,image,storage",
                         [(*s, *t) for s in SMALL for t in (TYPES if s[1] < 4 else TYPES[:1])])
def test_small_form_is_the_march_bitwise(rsf, shape, sigma, image, storage):
    """The small-volume form takes the march's sums in its order.  A split
    target makes the march run instead."""
    import torch
    I, phi0 = fields(shape, 13)
    if image == "u16":
        I = np.round(I * 65535.0).astype(np.uint16)
    p = rsf.make_params(sigma, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage)
    out = []
    with rsf.Context(0) as ctx:
        vol = torch.from_numpy(I).cuda()
        for waves in (0, 16):
            ctx.set_split_targets(waves, 0, 0)
            phi = torch.from_numpy(phi0).cuda()
            ctx.evolve_ex(vol, phi, p, 3)
            torch.cuda.synchronize()
            out.append(phi)
    assert torch.equal(out[1], out[0])
