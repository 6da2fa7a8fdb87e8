"""Work items of one to eight particles per thread in the particle pass and in
the reverse pass: all particles of a run in one tile, which the caller's item
size makes one item of 512, 513, 769, 3073 or 4096 particles (or two of half of
that), in a box that fits the LDS windows and in one as wide as the grid.  Against the
oracle, at the tolerances of the window tests of either pass."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import adjoint as oadj  # noqa: E402
from oracle import sipf as osipf  # noqa: E402
from test_gpu_adjoint_windows import rel  # noqa: E402
from test_gpu_particle_windows import _check  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402

SIZES = [(512, 4096), (513, 4096), (769, 4096), (1023, 512), (3073, 4096), (4096, 4096), (4097, 4096)]


def _largest(P, which, **prm):
    """Particles of the largest item when all are in one tile; the size rule has to leave the caller's."""
    got = pkg.dbg_plan([(prm, P)])[which]
    assert got == prm["chunk"]
    n = -(-P // got)
    return -(-P // n)


def _positions(P, wide, H):
    rng = np.random.default_rng(P + H)
    if wide:
        return rng.uniform(-1.0, 1.0, (P, 3))
    return rng.uniform(0.01, 0.49, (P, 3))  # within the tile of cells 8 .. 15 at H = 16


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("P,chunk", SIZES)
def test_particle_pass(precision, wide, P, chunk):
    H, tile = (32, 32) if wide else (16, 8)
    kw = dict(L=2.0, chi=3.0, mu=0.5, eps=1.0, k=1.0, M0=50.0, dt=1e-5, H=H, seed=11)
    size = _largest(P, "chunk", H=H, tile=tile, chunk=chunk, precision=precision)
    assert size == {1023: 512, 4097: 2049}.get(P, P)
    print("particle pass", precision, wide, P, size, flush=True)
    _check(precision, kw, _positions(P, wide, H), tile, chunk)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("P,chunk", SIZES)
def test_reverse_pass(precision, wide, P, chunk):
    H, tile = (32, 32) if wide else (16, 8)
    kw = dict(L=2.0, chi=1.5, mu=0.8, eps=1.0, k=1.0, M0=40.0, dt=1e-5, H=H, seed=21)
    size = _largest(P, "adj_chunk", H=H, tile=tile, chunk=chunk, precision=precision)
    print("reverse pass", precision, wide, P, size, flush=True)
    X0 = _positions(P, wide, H).astype(np.float32 if precision == "fp32" else np.float64)
    sim = pkg.Sim(X0, precision=precision, tile=tile, chunk=chunk, **kw)
    loss, dchi, dmu, dX0 = sim.adjoint(3, 3)
    ol, odX, ochi, omu = oadj.loss_and_grad(X0.astype(np.float64), osipf.Params(**kw), 3)
    tol = 1e-9 if precision == "fp64" else 1e-3
    assert abs(loss - ol) < tol * abs(ol)
    assert abs(dchi - ochi) < tol * max(abs(ochi), 1e-12)
    assert abs(dmu - omu) < tol * max(abs(omu), 1e-12)
    assert rel(dX0.cpu().numpy(), odX) < tol
    sim.close()


@pytest.mark.parametrize("P", [1500, 4096])
def test_reverse_pass_keeps_fp64(P):
    """One FP64 item whose gradient cotangents carry a quarter of the gradient (large chi).

    Rounding its 8 P terms at 2^-51 of the largest one changes the gradient by 7e-16, at 2^-51 of P times the
    largest by 2.7e-12 (P = 4096; planted in the oracle); the rest of the FP64 pass adds some 1e-14.
    """
    H = 16
    kw = dict(L=2.0, chi=200.0, mu=0.05, eps=1.0, k=1.0, M0=40.0, dt=1e-3, H=H, seed=21)
    assert _largest(P, "adj_chunk", H=H, tile=H, chunk=4096, precision="fp64") == P
    X0 = np.random.default_rng(1).uniform(-1.0, 1.0, (P, 3))
    sim = pkg.Sim(X0, precision="fp64", tile=H, chunk=4096, **kw)
    _, _, _, dX0 = sim.adjoint(3, 3)
    _, odX, _, _ = oadj.loss_and_grad(X0, osipf.Params(**kw), 3)
    err = rel(dX0.cpu().numpy(), odX)
    print(f"reverse pass FP64 P={P}: {err:.1e}", flush=True)
    assert err < 2e-13
    sim.close()
