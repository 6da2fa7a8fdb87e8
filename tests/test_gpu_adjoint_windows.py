"""Reverse particle pass where its LDS windows do not hold the item: tiles as
large as the grid, particles that drift out of their tile over a segment, noise
beyond the window's margin, grids smaller than a window, one particle, items of
the largest size.  Against the oracle adjoint at the tolerances of the adjoint
parity tests (FP64 1e-9, FP32 1e-3 relative)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import adjoint as oadj  # noqa: E402
from oracle import sipf as osipf  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300)


@pytest.mark.parametrize("precision,H,tile,P,chunk,N,K,dt,scheme", [
    ("fp64", 64, 64, 3001, 0, 3, 3, 1e-4, "strang"), ("fp64", 64, 64, 2001, 256, 3, 2, 1e-4, "em"),
    ("fp32", 64, 64, 5001, 0, 3, 3, 1e-4, "strang"), ("fp64", 32, 4, 4001, 512, 8, 8, 5e-4, "strang"),
    ("fp32", 64, 8, 5001, 0, 6, 6, 5e-4, "strang"), ("fp64", 32, 16, 2001, 0, 2, 2, 1e-2, "strang"),
    ("fp64", 8, 8, 4097, 4096, 3, 3, 1e-4, "strang"), ("fp64", 16, 16, 4096, 4096, 2, 1, 1e-4, "em"),
    ("fp32", 16, 16, 4500, 4096, 2, 2, 1e-4, "strang"), ("fp64", 16, 2, 1, 0, 2, 2, 1e-4, "strang")])
def test_adjoint_windows(precision, H, tile, P, chunk, N, K, dt, scheme):
    print("adjoint windows", precision, H, tile, P, chunk, N, K, dt, scheme, flush=True)
    kw = dict(L=2.0, chi=1.5, mu=0.8, eps=1.0, k=1.0, M0=40.0, dt=dt, H=H, seed=21, scheme=scheme)
    X0 = osipf.wrap(np.random.default_rng(P + H).normal(0.0, 0.4, (P, 3)), 2.0)
    X0 = X0.astype(np.float32 if precision == "fp32" else np.float64)
    sim = pkg.Sim(X0, precision=precision, tile=tile, chunk=chunk, **kw)
    loss, dchi, dmu, dX0 = sim.adjoint(N, K)
    ol, odX, ochi, omu = oadj.loss_and_grad(X0.astype(np.float64), osipf.Params(**kw), N)
    tol = 1e-9 if precision == "fp64" else 1e-3
    print(f" loss {abs(loss - ol) / abs(ol):.1e} chi {abs(dchi - ochi) / abs(ochi):.1e} mu "
          f"{abs(dmu - omu) / abs(omu):.1e} X0 {rel(dX0.cpu().numpy(), odX):.1e}", flush=True)
    assert abs(loss - ol) < tol * abs(ol)
    assert abs(dchi - ochi) < tol * max(abs(ochi), 1e-12)
    assert abs(dmu - omu) < tol * max(abs(omu), 1e-12)
    assert rel(dX0.cpu().numpy(), odX) < tol
    sim.close()
