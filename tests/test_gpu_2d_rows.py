"""Two-dimensional field passes at the grid sizes where their transforms and
layouts change (register and LDS stages, blocks of frequencies, the last block
partial): one step from a state with a gradient, and rho_max, against the FP64
oracle.  Tolerances of the 2-D step tests: FP32 2e-5 relative L2 in alpha and
the gradient grids, FP64 1e-11; rho_max 2e-5 and 1e-10 relative."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import diagnostics as odiag  # noqa: E402
from oracle import sipf as osipf  # noqa: E402
from oracle import sipf2d as o2  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402
from paper_2512_03452_amd import workloads  # noqa: E402


def rel_l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("H", [16, 32, 128, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_2d_fields(H, precision):
    print("2-D fields", H, precision, flush=True)
    kw = dict(L=8.0, chi=1.0, mu=1.0, eps=0.5, k=0.3, M0=30.0, dt=1e-3, H=H, seed=4)
    prm = osipf.Params(**kw)
    X0 = workloads.disk(3000, 1.0, seed=H).astype(np.float32 if precision == "fp32" else np.float64)
    sim = pkg.Sim(X0, dim=2, precision=precision, **kw)
    sim.run(2)
    X = sim.positions().cpu().numpy().astype(np.float64)
    A = sim.field("alpha").cpu().numpy().astype(np.complex128)
    sim.run(1)
    _, ao = o2.step(X, o2.full_spectrum(A), 3, prm)
    tol = 2e-5 if precision == "fp32" else 1e-11
    A3 = sim.field("alpha").cpu().numpy().astype(np.complex128)
    assert rel_l2(A3, o2.half_spectrum(ao)) < tol
    assert rel_l2(sim.field("grad").cpu().numpy().astype(np.float64), o2.gradient_grid(ao, prm)) < tol
    d = sim.diagnostics()
    want = odiag.all_diagnostics(sim.positions().cpu().numpy().astype(np.float64), o2.full_spectrum(A3), prm)
    rtol = 2e-5 if precision == "fp32" else 1e-10
    assert abs(d["rho_max"] - want["rho_max"]) < rtol * abs(want["rho_max"])
    assert abs(d["hf_share"] - want["hf_share"]) < rtol
    sim.close()
