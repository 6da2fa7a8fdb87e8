"""What the library chooses before it runs (sipf_dbg_plan): a work-item size that
the caller gives is taken as it is, in both passes, and left open it follows the
particle count."""

import pytest

pytest.importorskip("torch")

from paper_2512_03452_amd import _lib  # noqa: E402
from paper_2512_03452_amd.sim import dbg_plan  # noqa: E402


@pytest.mark.parametrize("chunk", [256, 513, 1024, 3072, 4096])
@pytest.mark.parametrize("H,P,dim", [(16, 500, 3), (46, 97336, 3), (64, 10 ** 6, 3), (128, 10 ** 7, 3), (64, 4097, 2)])
def test_given_item_size_is_taken(chunk, H, P, dim):
    p = dbg_plan([(dict(H=H, dim=dim, chunk=chunk), P)])
    assert p["chunk"] == chunk and p["adj_chunk"] == chunk
    # a batch takes the first instance's
    p = dbg_plan([(dict(H=H, dim=dim, chunk=chunk), P), (dict(H=H, dim=dim), P)])
    assert p["chunk"] == chunk


@pytest.mark.parametrize("P,chunk,adj", [(500, 256, 256), (97336, 512, 512), (2 * 10 ** 5, 1024, 1024),
                                         (10 ** 6, 3072, 4096), (10 ** 7, 4096, 4096)])
def test_item_size_left_open(P, chunk, adj):
    p = dbg_plan([(dict(H=64), P)])
    assert p["chunk"] == chunk and p["adj_chunk"] == adj
    assert dbg_plan([(dict(H=64, dim=2), P)])["chunk"] == 4096


def test_sizes_of_the_tuner_are_four_different_plans():
    plans = [dbg_plan([(dict(H=32, chunk=c), 40000)])["chunk"] for c in (1024, 2048, 3072, 4096)]
    assert plans == [1024, 2048, 3072, 4096]


def test_tiles_of_the_finest_grid():
    big, small = (dict(H=256), 1 << 18), (dict(H=32), 5000)
    assert dbg_plan([big]) == dict(dbg_plan([big]), keys=32768, tile=[8])
    assert dbg_plan([small, big]) == dict(dbg_plan([small, big]), keys=32768, tile=[8, 8])
    few = dbg_plan([(dict(H=256), (1 << 18) - 1)])
    assert few["keys"] == 4096 and few["tile"] == [16]
    assert dbg_plan([(dict(H=256, tile=16), 1 << 20)])["keys"] == 4096


def test_invalid_arguments():
    lib = _lib.load()
    assert lib.sipf_dbg_plan(1, None, None, None) == _lib.SIPF_EINVAL
    with pytest.raises(_lib.SipfError):
        dbg_plan([(dict(H=48), 100)])
    with pytest.raises(_lib.SipfError):
        dbg_plan([(dict(H=16, method="direct"), 100)])
