"""Gauge sweeps where the tests of test_gpu_gauge.py and test_gpu_edges.py do not go: links that are not exactly
SU(3), and launches of more than eight blocks with a remainder.  Tolerances as there: 1e-11 after one heatbath sweep
(the transcendental functions of the device and of the host library differ in the last bits), ten times that after a
further over-relaxation sweep."""
import numpy as np
import pytest

import dwfgen
from oracle import gauge as G

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _compare(U0, dims, n_or, tol):
    import paper_2602_14454_amd as dwf
    Ud = _dev(U0)
    dwf.gauge_sweeps(Ud, dims, 6.0, nsweeps=1, n_or=n_or, seed=77, sweep0=3)
    Uo = U0.copy()
    G.sweep(Uo, dims, 6.0, 77, 3, heatbath=True)
    for _ in range(n_or):
        G.sweep(Uo, dims, 6.0, 77, 3, heatbath=False)
    assert np.abs(Ud.cpu().numpy() - Uo).max() < tol


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 2, 6)])
@pytest.mark.parametrize("links", ["complex64", "off by 1e-3"])
def test_links_that_are_not_su3(dims, links):
    """The links are projected onto SU(3) after a sweep, not within it: the staples of a sweep see its own
    unprojected links."""
    U0 = dwfgen.random_su3_links(dims, 0.5, 5)
    if links == "complex64":
        U0 = U0.astype(np.complex64).astype(np.complex128)
    else:
        rng = np.random.default_rng(2)
        U0 = U0 + 1e-3 * (rng.standard_normal(U0.shape) + 1j * rng.standard_normal(U0.shape))
    _compare(U0, dims, 0, 1e-11)
    _compare(U0, dims, 1, 1e-10)


# 648 site pairs: 11 update blocks (8 XCDs and a remainder of 3), 20 whole tiles and one of 8 pairs; 360 pairs: 6 blocks
@pytest.mark.parametrize("dims", [(6, 6, 6, 6), (6, 6, 2, 10)])
def test_blocks_over_all_xcds(dims):
    U0 = dwfgen.random_su3_links(dims, 0.5, 5)
    _compare(U0, dims, 0, 1e-11)
    _compare(U0, dims, 1, 1e-10)
