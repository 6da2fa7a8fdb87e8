"""Reading alpha back: a spectrum given to sipf_init comes back bit for bit,
whatever the grid's storage order, through each route of sipf_get_field: an
aligned device buffer, a device buffer that is not aligned for whole complex
values, and host memory.  The values are copied, so the tolerance is zero."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU containers
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2512_03452_amd as pkg  # noqa: E402
from paper_2512_03452_amd import _lib  # noqa: E402


@pytest.mark.parametrize("dim,H,precision,method", [
    (3, 8, "fp32", "pic"), (3, 22, "fp32", "pic"), (3, 46, "fp64", "pic"), (3, 128, "fp32", "pic"),
    (3, 256, "fp32", "pic"), (2, 8, "fp32", "pic"), (2, 64, "fp64", "pic"), (2, 512, "fp32", "pic"),
    (2, 2048, "fp32", "pic"), (3, 12, "fp64", "direct")])
def test_alpha_comes_back_as_given(dim, H, precision, method):
    print(f"alpha read-back: dim={dim} H={H} {precision} {method}", flush=True)
    rdt = np.float32 if precision == "fp32" else np.float64
    rng = np.random.default_rng(H + dim)
    shape = (H,) * (dim - 1) + (H // 2 + 1,)
    grid = rng.normal(size=(H,) * dim)
    alpha = np.fft.rfftn(grid).astype(np.complex64 if precision == "fp32" else np.complex128)
    assert alpha.shape == shape
    X0 = rng.uniform(-0.5, 0.5, (10, dim)).astype(rdt)
    sim = pkg.Sim(X0, alpha0=alpha, precision=precision, H=H, dim=dim, method=method)
    got = sim.field("alpha").cpu().numpy()
    assert np.array_equal(got, alpha)
    lib = _lib.load()
    host = np.empty(2 * alpha.size, dtype=rdt)
    _lib.check(lib.sipf_get_field(sim._h, _lib.SIPF_FIELD_ALPHA, host.ctypes.data_as(ctypes.c_void_p), 0))
    assert np.array_equal(host.view(alpha.dtype).reshape(shape), alpha)
    odd = torch.zeros(2 * alpha.size + 1, dtype=torch.float32 if precision == "fp32" else torch.float64, device="cuda")
    _lib.check(lib.sipf_get_field(sim._h, _lib.SIPF_FIELD_ALPHA, ctypes.c_void_p(odd[1:].data_ptr()), 1))
    got = odd[1:].cpu().numpy().view(alpha.dtype).reshape(shape)
    assert np.array_equal(got, alpha) and float(odd[0]) == 0.0
    sim.close()
