"""Autotuning one small volume: its untuned splits (short chunks, the small form
of the xy pass) are not among those that workgroup targets give, and stay."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 64, 64), (45, 71, 67)])
def test_tuned_is_not_slower_than_untuned(shape):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2404_02813_amd import rsf
    rng = np.random.Generator(np.random.PCG64(31))
    vol = torch.from_numpy(rng.uniform(0.0, 1.0, shape).astype(np.float32)).cuda()
    phi0 = torch.from_numpy(rng.uniform(-3.0, 3.0, shape).astype(np.float32)).cuda()
    p = rsf.make_params(3.0, 1.0, 1.0, 0.001, 1.0, 0.1, 1.0)
    out, best = [], []
    with rsf.Context(0) as ctx, rsf.Context(0) as tuned:
        tuned.autotune([vol], [phi0], p)
        for c in (ctx, tuned):
            phi = phi0.clone()
            c.evolve_ex(vol, phi, p, 5)
            out.append(phi)
        for c in (ctx, tuned):
            least = float("inf")
            for _ in range(8):
                phi = phi0.clone()
                torch.cuda.synchronize()
                t = time.perf_counter()
                c.evolve_ex(vol, phi, p, 60)
                torch.cuda.synchronize()
                least = min(least, time.perf_counter() - t)
            best.append(least)
    assert torch.equal(out[0], out[1])
    # the least of eight: the candidates' best takes 1.3 to 1.6 times as long
    assert best[1] <= 1.15 * best[0]
