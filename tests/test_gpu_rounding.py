"""phi of a few iterations bit for bit: how the update's sums are rounded is part
of its result and must not move with the code around them (registers, unrolling,
fusion).  The CRCs below are of phi after three iterations of the same inputs
with the passes that came before the merged xy pass."""
import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE, ITERS = (21, 11, 67), 3

# (image, storage, force) -> CRC-32 of phi at radius 1, 2, .. 16 (FP32 fields of an
# FP32 image) or 4, 5, .. 12
CRC = {
    ("f32", "f32", "rsf"): [
        0xfcd8e9fd, 0x77f1dc40, 0xa3ca0d5b, 0x411b910d, 0x0760d998, 0xe6eac4a2,
        0x266a36d9, 0xad100367, 0x602005ae, 0xb610520e, 0x04f21b97, 0xa94bd735,
        0x63d58c5e, 0x3c4c0e65, 0xd66056c2, 0xe8077561,
    ],
    ("f32", "f32", "paper"): [
        0xadb4c8f6, 0xbe8f2890, 0xbfadbd0e, 0x98fbf5fd, 0x67cdb769, 0xc5114916,
        0x992edad4, 0x85353c6f, 0xadfd9f13, 0x023f916c, 0x168d6a65, 0xd2f81228,
        0xfefad4b7, 0x5e65ecdd, 0x2dd4a468, 0x7dc20b39,
    ],
    ("u16", "f32", "rsf"): [
        0x161543ad, 0xfb73b6e3, 0x10cf61ff, 0x4fa6baf4, 0xaabaeb1d, 0x7933a621,
        0x5aaf9e8b, 0xc53b3dea, 0xb6f3c029,
    ],
    ("u16", "f32", "paper"): [
        0x465b5898, 0xbdec7214, 0x6431f443, 0x22d1aa90, 0xecb8befa, 0xcc7601a3,
        0x0f2d57bb, 0x750f42ac, 0x68bbeba6,
    ],
    ("f32", "f16", "rsf"): [
        0xb1872e48, 0x45a11bf1, 0x4d8d5d17, 0x9fb4b047, 0x4aa8bbdf, 0x44575daf,
        0x1f74caf0, 0x584b71cf, 0x70f30ed5,
    ],
    ("f32", "f16", "paper"): [
        0x15993bb4, 0x7948c149, 0xd8db066f, 0x4b3e1888, 0x18de0d44, 0x730ca13c,
        0x40be3704, 0x02a3e937, 0x77552e1a,
    ],
    ("u16", "f16", "rsf"): [
        0x15321af6, 0xaeb735fe, 0x66b9e808, 0x34f90b94, 0x8af1cab7, 0x212dbef5,
        0x0363c6c2, 0x26ee4cdd, 0xc102f56e,
    ],
    ("u16", "f16", "paper"): [
        0x07aa8a88, 0x612fcf8e, 0x70e5849a, 0x0d3c5e8e, 0x274cb2c9, 0xaa7bfb2c,
        0x3b4d47f4, 0x880b8315, 0x58f3deec,
    ],
    ("f32", "bf16", "rsf"): [
        0xb0be7089, 0x146852fe, 0x9dac1b92, 0x1bcd39f4, 0xe9602438, 0xa215f61d,
        0xb3e3fa33, 0xced4787b, 0x12a9eaad,
    ],
    ("f32", "bf16", "paper"): [
        0x1888f556, 0x180a65fc, 0xabe11dc2, 0xb4785f82, 0x811201c0, 0xc79ac4d3,
        0xa89e0753, 0x0a54ba94, 0xfba15398,
    ],
    ("u16", "bf16", "rsf"): [
        0xe3285374, 0x0f481bfa, 0xc9e48b36, 0x9f2a5a41, 0x958f0755, 0xcd40a2eb,
        0x6483280c, 0x893fa9a7, 0x2e44b735,
    ],
    ("u16", "bf16", "paper"): [
        0x37fe3e23, 0xe2274e2d, 0x743f2e25, 0x910a9b88, 0x399fc418, 0xa4831448,
        0x40ac9f3d, 0x591ca1b2, 0xed25a30a,
    ],
}


def first_radius(key):
    return 1 if key[:2] == ("f32", "f32") else 4


def evolve(rsf, key, radius, fuse, iters=ITERS):
    import torch
    image, storage, force = key
    rng = np.random.Generator(np.random.PCG64(23))
    I = rng.uniform(0.0, 1.0, SHAPE).astype(np.float32)
    if image == "u16":
        I = np.round(I * 65535.0).astype(np.uint16)
    phi = torch.from_numpy(rng.uniform(-3.0, 3.0, SHAPE).astype(np.float32)).cuda()
    f = rsf.RSF_FORCE_PAPER if force == "paper" else rsf.RSF_FORCE_RSF
    p = rsf.make_params(radius / 3 - 0.05, 1.0, 1.5, 0.001, 1.0, 0.1, 1.0, storage=storage, force=f)
    with rsf.Context(0) as ctx:
        ctx.set_split_targets(0, 0, 1)   # the update whole in z, which lets it fuse
        ctx.set_fusion(fuse)
        ctx.evolve_ex(torch.from_numpy(I).cuda(), phi, p, iters)
        torch.cuda.synchronize()
    return zlib.crc32(phi.cpu().numpy().tobytes())


@pytest.mark.parametrize("fuse", [False, True])
@pytest.mark.parametrize("key", CRC, ids="-".join)
def test_phi_is_bitwise_what_it_was(key, fuse):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf
    r0 = first_radius(key)
    got = [evolve(rsf, key, r0 + k, fuse) for k in range(len(CRC[key]))]
    wrong = [r0 + k for k, c in enumerate(CRC[key]) if got[k] != c]
    assert not wrong, f"radii {wrong}"
