"""Which configurations lb_init takes: limits that are checked before any memory
is asked for (no GPU needed; with one, the allocator hook refuses everything)."""
import ctypes as ct

import pytest

from paper_0809_4958_amd import lbm


def init_status(boxes, storage, streaming):
    """lb_init's status with an allocator that has no memory to give."""
    lib = lbm.load()
    arr = (lbm.LbBox * len(boxes))(*[lbm.LbBox(*b, 0) for b in boxes])
    cfg = lbm.LbConfig(n_boxes=len(boxes), boxes=ct.cast(arr, ct.POINTER(lbm.LbBox)), collision=lbm.MRT, tau=0.8,
                       tau_bulk=0.8, ghost_rate=1.0, storage=storage, rho0=1.0, streaming=streaming,
                       dev_alloc=lbm.ALLOC_FN(lambda n, user: None), dev_free=lbm.FREE_FN(lambda p, user: None))
    h = ct.c_void_p()
    st = lib.lb_init(ct.byref(cfg), ct.byref(h))
    assert st != lbm.OK and not h.value
    return st


@pytest.mark.parametrize("nx,streaming,refused", [
    (8, lbm.STREAM_AB, True),    # rows of whole lane vectors: x-face velocities past 32-bit offsets
    (8, lbm.STREAM_AA, False),   # in place tile items do without
    (9, lbm.STREAM_AB, False),   # so do rows that would have to be padded
    (9, lbm.STREAM_AA, False)])
def test_x_face_offsets_refuse_only_rows_that_need_them(nx, streaming, refused):
    st = init_status([(nx, 4096, 4096)] * 22, lbm.STORE_F16DEV, streaming)
    assert (st == lbm.ERR_ARG) == refused, st
    assert refused or st in (lbm.ERR_OOM, lbm.ERR_HIP)
