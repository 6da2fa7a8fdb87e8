"""Sorts into many tiles: work items that share sparse tiles (H = 128 with a few
particles per tile, H/tile above and at the smallest tile counts that share),
the 32 tiles per axis of H = 256, and a batch that mixes them with a small
grid.  Against the oracle, at the tolerances of the particle window tests."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import sipf as osipf  # noqa: E402
from test_gpu_particle_windows import _check  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402


def _mixture(P, seed):
    # half uniform (a few per tile), half in a ball (full tiles)
    rng = np.random.default_rng(seed)
    return np.concatenate([rng.uniform(-1.0, 1.0, (P // 2, 3)), rng.normal(0.1, 0.1, (P - P // 2, 3))])


@pytest.mark.parametrize("precision,H,P,tile,scheme,pp", [
    ("fp32", 128, 20001, 0, "strang", "two_phase"), ("fp32", 128, 20001, 16, "strang", "two_phase"),
    ("fp32", 128, 9001, 0, "em", "sorted"), ("fp64", 64, 9001, 4, "strang", "default"),
    ("fp64", 64, 20001, 4, "em", "default"), ("fp32", 90, 20001, 6, "strang", "two_phase"),
    ("fp32", 256, (1 << 18) - 1, 0, "em", "two_phase"), ("fp32", 256, (1 << 18) + 1, 0, "em", "two_phase"),
    ("fp32", 256, (1 << 18) + 3, 0, "strang", "sorted")])
def test_sparse_tiles(precision, H, P, tile, scheme, pp):
    print("sparse tiles", precision, H, P, tile, scheme, pp, flush=True)
    kw = dict(L=2.0, chi=3.0, mu=0.05, eps=1.0, k=1.0, M0=50.0, dt=1e-4, H=H, seed=13, scheme=scheme)
    _check(precision, kw, _mixture(P, H + P), tile, 0, steps=3 if H < 256 else 1, resort=2, particle_pass=pp)


def test_batch_of_many_and_few_tiles():
    # every instance of a batch is sorted with the largest instance's key count
    kw = dict(L=2.0, chi=3.0, mu=0.05, eps=1.0, k=1.0, M0=50.0, dt=1e-4, seed=17)
    grids, counts = [16, 256, 46], [5001, (1 << 18) + 1, 3001]
    X0 = [_mixture(P, H).astype(np.float32) for H, P in zip(grids, counts)]
    batch = pkg.Batch([dict(X0=x, params=dict(kw, H=H, precision="fp32", instance=i))
                       for i, (x, H) in enumerate(zip(X0, grids))])
    batch.run(13)
    for i, (x, H) in enumerate(zip(X0, grids)):
        sim = pkg.Sim(x, precision="fp32", tile=16 if H == 256 else 0, instance=i, **dict(kw, H=H))
        sim.run(13)
        d = batch.positions(i).cpu().numpy().astype(np.float64) - sim.positions().cpu().numpy()
        err = np.abs(osipf.min_image(d, 2.0)).max()
        print(f"batch instance {i} H={H}: {err:.2e}", flush=True)
        assert err < 2 * 13 * 1e-6  # 13 steps of either run's single-step bound (the drift's part is far below it)
        sim.close()
    batch.close()
