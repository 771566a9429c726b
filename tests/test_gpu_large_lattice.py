"""Tables and fields beyond 4 GiB, past what a 32-bit byte offset addresses.

48^3 x 68 has 3.76 M sites per parity: the FP64 link table of one parity has 4.33 GB, the FP32 one 2.41 GB.
"""
import gc

import pytest

pytestmark = pytest.mark.gpu

DIMS = (48, 48, 48, 68)


@pytest.fixture(scope="module")
def lattice():
    import torch

    import paper_2602_14454_amd as dwf
    lat = dwf.Lattice(DIMS)
    g = torch.Generator(device="cuda").manual_seed(3)
    # every link different (the hop is linear in them and needs no SU(3))
    U = torch.randn((lat.V, 4, 3, 3, 2), dtype=torch.float64, device="cuda", generator=g)
    lat.set_gauge(torch.view_as_complex(U))
    del U
    torch.cuda.empty_cache()
    yield lat
    del lat
    gc.collect()
    torch.cuda.empty_cache()


def test_link_table_beyond_4gib(lattice):
    """FP64 D^ with the large table against FP32, whose table is below the limit; FP32 tolerance of
    test_gpu_operator.py."""
    import torch

    import paper_2602_14454_amd as dwf
    op = dwf.Op(lattice, 2, 1.6, 0.05, 1.0, 0.0, 0.6)
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((2, lattice.Vh, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    a, b = torch.empty_like(x), torch.empty_like(x)
    op.apply(a, x, dwf.EVEN5D, False, 0)
    op.apply(b, x, dwf.EVEN5D, False, 1)
    assert float((a - b).abs().max() / a.abs().max()) < 1e-5


def test_residual_update_beyond_4gib(lattice):
    """r -= alpha D^dag D^ p with BF16 fields of 2.17 GB and an FP32 r of 4.33 GB: against the normal operator, whose
    result is rounded to BF16 (2^-9 of its largest entry)."""
    import torch

    import paper_2602_14454_amd as dwf
    op = dwf.Op(lattice, 12, 1.6, 0.05, 1.0, 0.0, 0.6)
    g = torch.Generator(device="cuda").manual_seed(5)
    p = torch.randn((12, lattice.Vh, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    w = torch.empty_like(p)
    op.apply_normal(w, p, 2)
    r = torch.zeros_like(p)
    r[:, ::7] = p[:, ::7]   # alpha = |r|^2 / |D^ p|^2 is not zero
    want = r.clone()
    alpha, rr = op.cg_residual_update(r, p, 2)
    assert alpha > 0.0
    want -= alpha * w
    scale = alpha * float(w.abs().max())
    assert float((r - want).abs().max()) < 4e-3 * scale
    assert abs(rr / float((torch.view_as_real(r) ** 2).sum()) - 1) < 1e-5
