"""Fast sweeping at the edges of its blocks (16 x 16 lines by
32 hyperplanes), against the FP64 oracle's sweep of the same seeds."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# (nz, ny, nx): the smallest volume, the fewest lines along each axis, one block's
# lines and one less and more, several blocks with remainders, rows
# shorter than the skew and longer than a wave
SHAPES = [(3, 3, 3), (3, 3, 70), (3, 40, 3), (70, 3, 3), (31, 15, 9), (32, 16, 16), (33, 17, 65),
          (65, 33, 4), (3, 49, 130), (66, 3, 5)]


@pytest.mark.parametrize("rounds", [1, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_sweep_matches_the_oracle(shape, rounds):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf
    rng = np.random.Generator(np.random.PCG64(5))
    n = int(np.prod(shape))
    u0 = np.full(n, oracle.FAR)
    u0[rng.choice(n, size=min(n, 5), replace=False)] = 0.0
    u0 = u0.reshape(shape)
    u = torch.from_numpy(u0.astype(np.float32)).cuda()
    with rsf.Context(0) as ctx:
        ctx.fast_sweep(u, rounds)
        torch.cuda.synchronize()
    want = oracle.fast_sweep(u0, rounds)
    # FP32 distances: 2^-24 per update along a path of up to 130 voxels
    assert np.all(np.abs(u.cpu().numpy() - want) <= 1e-5 + 1e-5 * want)
