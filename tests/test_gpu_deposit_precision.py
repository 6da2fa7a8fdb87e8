"""The FP32 deposit where few particles spread over many nodes: items of less
than 64 particles, items that share sparse tiles, boxes wider than the window, the
tiles of H = 256.  The density at the context's own positions against its deposit
in 64 bits, relative L2.

Bound: an FP32 weight is a product of about eight rounded factors, 5e-8 rms; its
sum takes one rounding per window that reaches the node (two or three of 2^-24
each).  2 x 2^-24 where a node meets a few particles, 4 x 2^-24 where the windows
of neighbouring items add up in FP32.  Weights rounded at a scale for the whole
item's count on one node are two to fifteen times further off."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import sipf as osipf  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402

ULP = 2.0 ** -24


def _positions(kind, P):
    rng = np.random.default_rng(P)
    if kind == "uniform":
        return rng.uniform(-1.0, 1.0, (P, 3))
    t, a = 2 * np.pi * rng.random(P), 0.05 * rng.normal(size=(P, 2))
    return np.stack([(0.5 + a[:, 0]) * np.cos(t), (0.5 + a[:, 0]) * np.sin(t), a[:, 1]], axis=1)


@pytest.mark.parametrize("kind,H,P,tile,steps,pp,ulps", [
    ("uniform", 32, 10001, 0, 0, "two_phase", 2), ("uniform", 64, 20001, 0, 5, "two_phase", 2),
    ("uniform", 64, 20001, 0, 5, "sorted", 2), ("uniform", 128, 50001, 0, 0, "two_phase", 2),
    ("uniform", 128, 50001, 0, 5, "sorted", 2), ("uniform", 64, 50001, 64, 0, "two_phase", 4),
    ("torus", 128, 20001, 32, 3, "two_phase", 4), ("torus", 256, 200001, 0, 5, "two_phase", 4),
    ("torus", 256, 300001, 0, 5, "two_phase", 4)])
def test_deposit_keeps_fp32_weights(kind, H, P, tile, steps, pp, ulps):
    print("deposit precision", kind, H, P, tile, steps, pp, flush=True)
    kw = dict(L=2.0, chi=1.0, mu=1.0, eps=1.0, k=1.0, M0=60.0, dt=5e-5, H=H, seed=3)
    X0 = osipf.wrap(_positions(kind, P), 2.0).astype(np.float32)
    sim = pkg.Sim(X0, precision="fp32", tile=tile, particle_pass=pp, **kw)
    sim.run(steps)
    X = sim.positions().cpu().numpy().astype(np.float64)
    rho = sim.field("rho").cpu().numpy().astype(np.float64)
    exact = osipf.deposit(X, 60.0 / P, H, 2.0, 4)
    err = np.linalg.norm(rho - exact) / np.linalg.norm(exact)
    print(f" error {err:.2e} (bound {ulps * ULP:.2e})", flush=True)
    assert err < ulps * ULP
    sim.close()


@pytest.mark.parametrize("H,P,tile", [(8, 700, 8), (12, 1400, 12), (16, 1023, 16), (64, 1400, 64)])
def test_fp64_deposit_keeps_its_bits(H, P, tile):
    """FP64 items of 513 to 1489 particles on small grids and in wide boxes, against extended precision.

    Weights carry about eight roundings of half a unit of 2^-53 relative, and are then rounded at 2^-52 or finer
    (2^-53 of a weight's unit, rms 2^-54.8): with n weights of about 0.1 on a node, sqrt(n) (0.29 x 2^-52 + 1e-17),
    and the sum itself is rounded twice.  A scale of 2^50 is four times coarser.
    """
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision")
    print("fp64 deposit", H, P, tile, flush=True)
    X0 = np.random.default_rng(P).uniform(-1.0, 1.0, (P, 3))
    assert pkg.dbg_plan([(dict(H=H, tile=tile, chunk=4096, precision="fp64"), P)])["chunk"] == 4096  # one item
    sim = pkg.Sim(X0, precision="fp64", tile=tile, chunk=4096, L=2.0, chi=1.0, mu=1.0, eps=1.0, k=1.0, M0=float(P), dt=5e-5, H=H,
                  seed=3)
    X = sim.positions().cpu().numpy()
    rho = sim.field("rho").cpu().numpy()
    sim.close()
    ld = np.longdouble
    s = (X * (H / 2.0)).astype(ld)  # in cells, as rounded in FP64: the weights and sums are what is measured
    g = np.floor(s)
    lam = s - g
    g = g.astype(np.int64)
    om = 1 - lam
    lo = lam * om
    w = [-(2 - lam) * lo / 6, om, lam, -(1 + lam) * lo / 6]
    S = 1 + lo.sum(axis=1) / 2
    exact, count = np.zeros(H ** 3, dtype=ld), np.zeros(H ** 3)
    for i in range(4):
        for j in range(4):
            for k in range(4):
                outer = (i in (0, 3)) + (j in (0, 3)) + (k in (0, 3))
                if outer > 1:
                    continue
                F = w[i][:, 0] * w[j][:, 1] * w[k][:, 2] * (S if outer == 0 else 1)
                node = (((g[:, 0] - 1 + i) % H) * H + (g[:, 1] - 1 + j) % H) * H + (g[:, 2] - 1 + k) % H
                np.add.at(exact, node, F)
                np.add.at(count, node, 1.0)
    err = np.sqrt(np.mean(((rho.ravel().astype(ld) - exact) ** 2).astype(np.float64)))
    n, total = count.mean(), np.sqrt(np.mean((exact ** 2).astype(np.float64)))
    bound = np.sqrt(n) * (0.29 * 2.0 ** -52 + 1e-17) + 2 * 0.29 * 2.0 ** -53 * total
    coarse = np.sqrt(n) * 0.29 * 2.0 ** -50
    print(f" rms error {err:.2e} (bound {bound:.2e}; at 2^50 {coarse:.2e})", flush=True)
    assert err < bound
