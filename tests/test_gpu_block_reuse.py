"""Contexts on memory that an earlier context held: a smaller one on a block
of a larger one, a 2-D and a direct one after it, another stream, and the memory
given back by sipf_release_cached_memory.  Against the oracle, at the tolerances
of the particle window tests (a block's earlier contents must not show)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import sipf as osipf  # noqa: E402
from test_gpu_particle_windows import _check, rel_l2  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402
from paper_2512_03452_amd import _lib  # noqa: E402

KW = dict(L=2.0, chi=3.0, mu=0.5, eps=1.0, k=1.0, M0=50.0, dt=1e-3, seed=11)


def _release():
    _lib.check(_lib.load().sipf_release_cached_memory())


def _free():
    """Free device memory, what torch's own cache holds counted as free."""
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()


def _used_and_closed(P, H, stream=None, **kw):
    """A context whose buffers are all in use, closed again; the device memory it took."""
    rng = np.random.default_rng(P)
    before = _free()
    sim = pkg.Sim(rng.normal(0.0, 0.3, (P, 3)).astype(np.float32), H=H, stream=stream, **dict(KW, seed=99), **kw)
    taken = before - _free()
    sim.run(9)
    sim.diagnostics()
    sim.close()
    return taken


@pytest.mark.parametrize("precision,H,P", [("fp32", 32, 30001), ("fp64", 16, 9001), ("fp32", 46, 20001)])
def test_smaller_context_on_a_used_block(precision, H, P):
    print("used block", precision, H, P, flush=True)
    _release()
    rdt = 4 if precision == "fp32" else 8
    _used_and_closed(P * rdt // 4 * 5 // 4, H)
    X0 = np.random.default_rng(H).normal(0.0, 0.3, (P, 3))
    _check(precision, dict(KW, H=H), X0, 0, 0, steps=2)


def test_block_moves_to_another_stream():
    print("another stream", flush=True)
    _release()
    prm = dict(KW, H=32)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    X0 = np.random.default_rng(3).normal(0.0, 0.3, (20001, 3)).astype(np.float32)
    _used_and_closed(25001, 32, stream=a)
    sim = pkg.Sim(X0, stream=b, **prm)
    sim.step()
    Xo, ao = osipf.run(osipf.wrap(X0.astype(np.float64), 2.0), osipf.Params(**prm), 1)
    al = sim.field("alpha").cpu().numpy().astype(np.complex128)
    err = np.abs(osipf.min_image(sim.positions().cpu().numpy() - Xo, 2.0)).max()
    assert err < 1e-6
    assert rel_l2(al, osipf.half_spectrum(ao)) < 1e-5
    sim.close()


def test_closed_contexts_memory_is_kept_and_given_back():
    print("kept memory", flush=True)
    _release()
    taken = _used_and_closed(2000000, 64)
    assert taken >= 2000000 * 2 * 16
    kept = _free()
    assert _used_and_closed(2000000, 64) < taken // 8  # on the kept block
    _release()
    assert _free() - kept >= taken - (8 << 20)
    # 16 contexts of 120 MB at once: at most 1 GiB of them stays
    before = _free()
    sims = [pkg.Sim(np.zeros((3000000, 3), np.float32), H=64, **KW) for _ in range(16)]
    assert before - _free() > (3 << 29)
    for s in sims:
        s.close()
    assert before - _free() <= (1 << 30) + (64 << 20)
    _release()
