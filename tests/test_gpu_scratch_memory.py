"""Device memory that calls leave behind: shared by operators of one shape, bounded over all shapes, given back on
request and with the last operator."""
import gc

import pytest

pytestmark = pytest.mark.gpu


def _lattice(dims):
    import torch

    import paper_2602_14454_amd as dwf
    lat = dwf.Lattice(dims)
    lat.set_gauge(torch.eye(3, dtype=torch.complex128, device="cuda").expand(lat.V, 4, 3, 3).contiguous())
    return lat


def _op(lat, Ls, alpha=0.5):
    import paper_2602_14454_amd as dwf
    return dwf.Op(lat, Ls, 1.6, 0.05, 1.0, 0.0, alpha)


def _free():
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _normal(op):
    import torch
    x = torch.ones((op.Ls, op.lattice.Vh, 4, 3), dtype=torch.complex128, device="cuda")
    return op.apply_normal(torch.empty_like(x), x)


def test_operators_of_one_shape_share_it():
    """An alpha scan: six operators leave what one leaves (four half fields of 101 MB)."""
    lat = _lattice((16, 16, 16, 16))
    ops = [_op(lat, 16, 0.4 + 0.1 * k) for k in range(6)]
    _normal(ops[0])
    one = _free()
    for op in ops[1:]:
        _normal(op)
    assert one - _free() < 101e6


def test_release_and_last_operator_give_it_back():
    import torch

    import paper_2602_14454_amd as dwf
    lat = _lattice((16, 16, 16, 16))
    op, other = _op(lat, 16), _op(lat, 16, 0.7)
    dwf.release_scratch()
    before = _free()
    want = _normal(op).cpu()
    assert before - _free() > 390e6
    dwf.release_scratch()
    assert abs(before - _free()) < 64e6
    assert torch.equal(_normal(op).cpu(), want)
    del op
    assert before - _free() > 390e6   # the other operator may still use it
    del other
    assert before - _free() < 64e6


def test_bounded_over_all_shapes():
    """Eight shapes whose fields take 25 GB together leave no more than the 8 GiB that the header promises."""
    import paper_2602_14454_amd as dwf
    lat = _lattice((24, 24, 24, 48))
    ops = [_op(lat, Ls) for Ls in range(9, 17)]
    dwf.release_scratch()
    before = _free()
    for op in ops:
        _normal(op)
    assert before - _free() < (8 << 30) + 64e6
