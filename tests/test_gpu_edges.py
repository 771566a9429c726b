"""Kernels at the edges of their tiles, against the FP64 CPU oracle.

Tolerances as in test_gpu_operator.py: relative max-norm error FP64 1e-13,
FP32 1e-5, BF16 3e-2.
"""
import numpy as np
import pytest

import dwfgen
import oracle

pytestmark = pytest.mark.gpu

TOL = {0: 1e-13, 1: 1e-5, 2: 3e-2}


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _make(dims, Ls, seed=5, b=1.0, c=0.0, alpha=0.6):
    import paper_2602_14454_amd as dwf
    U = dwfgen.random_su3_links(dims, 0.5, seed)
    lat = dwf.Lattice(dims)
    lat.set_gauge(U)
    return lat, dwf.Op(lat, Ls, 1.6, 0.05, b, c, alpha), oracle.Params(dims=dims, Ls=Ls, M0=1.6, m=0.05, b=b, c=c, alpha=alpha), U


# sites per parity: 8 (part of a tile), 32 and 64 (one tile of the full and of
# the half conversion), 72 (remainder 8), 96, 120, 1008 (several bricks' rows)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 2, 4), (4, 4, 2, 4), (6, 6, 2, 2), (4, 6, 4, 2), (6, 10, 2, 2),
                                  (6, 6, 4, 14)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_layout_conversion_tiles(dims, prec):
    """Canonical <-> internal conversion of full and even vectors around the 64-site tiles."""
    import torch

    import paper_2602_14454_amd as dwf
    lat, op, p, U = _make(dims, 3)
    x = dwfgen.gaussian_source_5d(dims, 3, 9)
    out = torch.full(x.shape, float("nan"), dtype=torch.complex128, device="cuda")
    op.apply(out, _dev(x), dwf.FULL5D, False, prec)
    assert _rel(out.cpu().numpy(), oracle.dwf_apply(p, U, x)) < TOL[prec]
    xe = np.ascontiguousarray(x[:, : p.Vh])
    oe = torch.full(xe.shape, float("nan"), dtype=torch.complex128, device="cuda")
    op.apply(oe, _dev(xe), dwf.EVEN5D, True, prec)
    assert _rel(oe.cpu().numpy(), oracle.dhat(p, U, xe, dagger=True)) < TOL[prec]


# 8 and 24 sites per parity (part of a wave), 64, 72 and 1008; extents of 2 (both neighbours the same site)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 6, 2), (4, 4, 2, 4), (2, 6, 6, 2), (6, 6, 4, 14)])
@pytest.mark.parametrize("antiperiodic", [True, False])
def test_link_tables(dims, antiperiodic):
    """Links of host and device arrays, of a second configuration on the same lattice, in every precision."""
    import torch

    import paper_2602_14454_amd as dwf
    p = oracle.Params(dims=dims, Ls=2, M0=1.6, m=0.05, alpha=0.6, antiperiodic_t=int(antiperiodic))
    lat = dwf.Lattice(dims, antiperiodic)
    op = dwf.Op(lat, 2, 1.6, 0.05, 1.0, 0.0, 0.6)
    x = dwfgen.gaussian_source_5d(dims, 2, 4)
    out = torch.empty(x.shape, dtype=torch.complex128, device="cuda")
    for seed, host in ((1, True), (2, False), (3, True)):
        U = dwfgen.random_su3_links(dims, 0.7, seed)
        lat.set_gauge(U if host else _dev(U))
        want = oracle.dwf_apply(p, U, x)
        for prec in (0, 1, 2):
            op.apply(out, _dev(x), dwf.FULL5D, False, prec)
            assert _rel(out.cpu().numpy(), want) < TOL[prec]


def test_call_scratch_is_private_and_clean():
    """Scratch kept by an operator between calls: what earlier calls of other kinds left in it changes no
    result, and calls from two threads on two streams do not share it."""
    import threading

    import torch

    import paper_2602_14454_amd as dwf
    dims, Ls = (6, 6, 4, 14), 4
    lat, op, p, U = _make(dims, Ls)
    _, fresh, _, _ = _make(dims, Ls)
    V = p.V
    x5 = [_dev(dwfgen.gaussian_source_5d(dims, Ls, 20 + k)) for k in range(2)]
    out5 = torch.empty_like(x5[0])
    for prec in (0, 1, 2):
        op.apply(out5, x5[0], dwf.FULL5D, False, prec)
        op.apply_normal(out5[:, : V // 2].contiguous(), x5[0][:, : V // 2].contiguous(), prec)
    op.apply_eo5(out5, x5[0], False, 0)
    op.apply_eo5(out5, x5[0], True, 1)
    op.source_4d(out5, x5[0][0].contiguous())
    pvec = x5[1][:, : V // 2].contiguous()
    for prec in (0, 1, 2):
        got = []
        for o in (op, fresh):
            r = x5[0][:, : V // 2].contiguous()
            got.append((o.cg_residual_update(r, pvec, prec), r))
        assert got[0][0] == got[1][0] and torch.equal(got[0][1], got[1][1])
    assert op.true_residual(x5[0], x5[1]) == fresh.true_residual(x5[0], x5[1])

    want = [fresh.apply(torch.empty_like(x), x).clone() for x in x5]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        st = torch.cuda.Stream()
        out = torch.empty_like(x5[k])
        for _ in range(20):
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            op.apply(out, x5[k], stream=st.cuda_stream)
            if not torch.equal(out, want[k]):
                bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


# sites per parity 8 (a quarter of a 32-site tile), 32, 72 and 1008; every form of the hidden layer
@pytest.mark.parametrize("dims,Ls,H", [((2, 2, 2, 2), 2, 4), ((4, 4, 2, 2), 5, 1), ((6, 6, 2, 2), 16, 5),
                                       ((4, 2, 4, 2), 3, 3), ((6, 6, 4, 14), 2, 64)])
def test_network_tiles(dims, Ls, H):
    """Network output and weight gradient around the tiles and the number of hidden channels."""
    import torch

    import paper_2602_14454_amd as dwf
    from oracle import ptc as optc
    lat, op, p, U = _make(dims, Ls, alpha=0.5)
    W1, W2 = (w.astype(np.complex64).astype(np.complex128) for w in optc.random_weights(H, 5))
    M = dwf.PtcModel(H)
    M.set_weights(W1, W2)
    M.set_loss(0)
    r, e = (dwfgen.gaussian_source_5d(dims, Ls, k)[:, : p.Vh].astype(np.complex64).astype(np.complex128) for k in (6, 7))
    out = torch.full(r.shape, float("nan"), dtype=torch.complex128, device="cuda")
    M.apply(op, out, _dev(r))
    assert _rel(out.cpu().numpy(), optc.forward(U, dims, W1, W2, r)[0]) < 2e-5
    loss, grads = M.gradient(op, _dev(r), _dev(e))
    L, *want = optc.gradients(U, dims, W1, W2, r, e, kind=0)
    assert abs(loss - L) < 3e-5 * L
    for g, o in zip(grads, want):
        assert np.linalg.norm(g - o) < 3e-5 * np.linalg.norm(o)


@pytest.mark.parametrize("kind", [0, 1])
def test_network_on_two_lattices(kind):
    """One model on a large and then a smaller lattice gives what a new model gives on the small one."""
    import paper_2602_14454_amd as dwf
    from oracle import ptc as optc
    big, small = _make((6, 6, 4, 14), 4)[:2], _make((6, 2, 2, 6), 3)[:2]
    W = optc.random_weights(4, 5)
    got = []
    for ops in ((big, small), (small,)):
        M = dwf.PtcModel(4)
        M.set_weights(*W)
        M.set_loss(kind)
        for lat, op in ops:
            r, e = (_dev(np.ascontiguousarray(dwfgen.gaussian_source_5d(lat.dims, op.Ls, k)[:, : lat.Vh])) for k in (6, 7))
            loss, (g1, g2) = M.gradient(op, r, e)
        got.append((loss, g1, g2))
    assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])


# FP64 launches of 768 waves take the form for few blocks, of 784 and 896 the general one; Ls with a remainder
@pytest.mark.parametrize("dims,Ls", [((8, 8, 8, 12), 16), ((8, 8, 8, 14), 14), ((4, 14, 14, 8), 13), ((8, 8, 4, 6), 2)])
@pytest.mark.parametrize("b,c", [(1.0, 0.0), (1.5, 0.5)])
def test_hop_forms_by_lattice_size(dims, Ls, b, c):
    """Every kind of hop launch (plain, local term dense or not, two outputs, residual update) on both sides of
    the size rule, in FP64, and the specialised epilogues in FP32."""
    import torch

    import paper_2602_14454_amd as dwf
    lat, op, p, U = _make(dims, Ls, b=b, c=c)
    x = dwfgen.gaussian_source_5d(dims, Ls, 9)
    out = torch.empty(x.shape, dtype=torch.complex128, device="cuda")
    xe = np.ascontiguousarray(x[:, : p.Vh])
    oe = torch.empty(xe.shape, dtype=torch.complex128, device="cuda")
    q = oracle.dhat(p, U, xe)
    normal = oracle.dhat(p, U, q, dagger=True)
    for prec in (0, 1):
        for dagger in (False, True):
            op.apply(out, _dev(x), dwf.FULL5D, dagger, prec)
            assert _rel(out.cpu().numpy(), oracle.dwf_apply(p, U, x, dagger=dagger)) < TOL[prec]
        op.apply(oe, _dev(xe), dwf.EVEN5D, True, prec)
        assert _rel(oe.cpu().numpy(), oracle.dhat(p, U, xe, dagger=True)) < TOL[prec]
        op.apply_normal(oe, _dev(xe), prec)
        assert _rel(oe.cpu().numpy(), normal) < TOL[prec]
        r = _dev(np.ascontiguousarray(x[:, p.Vh:]))
        r0 = r.cpu().numpy()
        alpha, rr = op.cg_residual_update(r, _dev(xe), prec)
        want_a = np.linalg.norm(r0) ** 2 / np.linalg.norm(q) ** 2
        want = r0 - want_a * normal
        assert abs(alpha / want_a - 1) < TOL[prec]
        assert _rel(r.cpu().numpy(), want) < TOL[prec] and abs(rr / np.linalg.norm(want) ** 2 - 1) < TOL[prec]


# 8, 24, 80 and 144 site pairs: part of a 32-pair tile, remainders of several; extents of 2 and 10
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 6, 2, 2), (10, 2, 2, 4), (6, 2, 6, 4)])
def test_gauge_tiles(dims):
    """A heatbath and an over-relaxation sweep around the tiles of the working layout; tolerance of the
    single sweep in test_gpu_gauge.py, ten times for the second."""
    import paper_2602_14454_amd as dwf
    from oracle import gauge as G
    U0 = dwfgen.random_su3_links(dims, 0.5, 5)
    for n_or, tol in ((0, 1e-11), (1, 1e-10)):
        Ud = _dev(U0)
        dwf.gauge_sweeps(Ud, dims, 6.0, nsweeps=1, n_or=n_or, seed=77, sweep0=3)
        Uo = U0.copy()
        G.sweep(Uo, dims, 6.0, 77, 3, heatbath=True)
        for _ in range(n_or):
            G.sweep(Uo, dims, 6.0, 77, 3, heatbath=False)
        assert np.abs(Ud.cpu().numpy() - Uo).max() < tol
    Ud = _dev(U0)
    dwf.gauge_sweeps(Ud, dims, 6.0, nsweeps=0, n_or=2)
    assert np.array_equal(Ud.cpu().numpy(), U0)


# sites per parity 8 (part of a 64-site tile), 72 (remainder), 1008 (two tiles per XCD); slices of one parity 1 to 8
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((6, 6, 2, 2), 6), ((6, 6, 4, 14), 10), ((4, 2, 4, 2), 16)])
@pytest.mark.parametrize("prec", [0, 1])
def test_eo5_tiles(dims, Ls, prec):
    """Schur operator of the 5D split around its tiles: even entries against the oracle, odd ones zero."""
    import torch

    from oracle import eo5
    lat, op, p, U = _make(dims, Ls, alpha=0.6)
    x = dwfgen.gaussian_source_5d(dims, Ls, 9)
    odd = ~eo5.even_mask(p)
    for dagger in (False, True):
        out = torch.full(x.shape, float("nan"), dtype=torch.complex128, device="cuda")
        op.apply_eo5(out, _dev(x), dagger, prec)
        got = out.cpu().numpy()
        assert _rel(got, eo5.dhat5(p, U, x, dagger=dagger)) < TOL[prec] and np.all(got[odd] == 0)


# sites per parity 8 (half a tile of 16), 16, 24, 72 (remainder 8), 1008
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 2, 4), (2, 2, 6, 2), (6, 6, 2, 2), (6, 6, 4, 14)])
def test_neighbour_table_tiles(dims):
    """The device's neighbour table, read back through its tiles, names the sites next to each site."""
    import paper_2602_14454_amd as dwf
    lex, nbr = dwf.Lattice(dims).maps()
    step = np.cumprod((1,) + dims[:3])
    for d in range(8):
        mu, n = d % 4, dims[d % 4]
        c = lex // step[mu] % n
        assert np.array_equal(nbr[:, d], lex + ((c + (1 if d < 4 else -1)) % n - c) * step[mu])


def test_network_on_lattices_of_equal_tiles():
    """One model on 80 and then 72 sites per parity (both five tiles): the second lattice's padding is clean."""
    import paper_2602_14454_amd as dwf
    from oracle import ptc as optc
    first, second = _make((2, 2, 4, 10), 3)[:2], _make((6, 6, 2, 2), 3)[:2]
    W = optc.random_weights(4, 5)
    got = []
    for ops in ((first, second), (second,)):
        M = dwf.PtcModel(4)
        M.set_weights(*W)
        for lat, op in ops:
            r, e = (_dev(np.ascontiguousarray(dwfgen.gaussian_source_5d(lat.dims, op.Ls, k)[:, : lat.Vh])) for k in (6, 7))
            loss, (g1, g2) = M.gradient(op, r, e)
        got.append((loss, g1, g2))
    assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])


# 1, 9 and 256 partials (summed by the kernels that use them), 288 (by a kernel of its own); Ls = 4: always so
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 5), ((2, 6, 6, 4), 8), ((8, 8, 8, 16), 5), ((8, 8, 8, 18), 5),
                                     ((4, 4, 4, 4), 4)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_cg_scalars_by_lattice_size(dims, Ls, prec):
    """CG with its step lengths formed in the hop and in the p update: convergence to the oracle's residual
    for any check period."""
    import torch

    import paper_2602_14454_amd as dwf
    lat, op, p, U = _make(dims, Ls)
    b = dwfgen.gaussian_source_5d(dims, Ls, 12)
    x = torch.zeros(b.shape, dtype=torch.complex128, device="cuda")
    for check in (1, 3):
        prm = dwf.default_params(algo=dwf.ALGO_DC if prec else dwf.ALGO_CGNR, inner_prec=prec, check_every=check, tol=1e-10)
        x.zero_()
        st, info = op.solve(x, _dev(b), prm)
        assert st == 0 and info.converged
        assert oracle.true_residual(p, U, x.cpu().numpy(), b) <= 1.2e-10


# intermediate fields of 201 and 245 MB (plain stores) and 264 MB (non-temporal ones); Ls = 2, 3: every combination
# of missing neighbour slices
@pytest.mark.parametrize("dims,Ls", [((16, 16, 16, 16), 8), ((16, 16, 16, 12), 13), ((16, 16, 16, 12), 14),
                                     ((4, 4, 4, 4), 2), ((4, 4, 4, 4), 3)])
def test_network_sizes_against_layers(dims, Ls):
    """Two channels, of which the second is zero (pair sums), against the one channel (layer by layer): the same
    sums in FP32, whose rounding is below 1e-6 of a field in either."""
    import torch

    import paper_2602_14454_amd as dwf
    from oracle import ptc as optc
    lat = dwf.Lattice(dims)
    g = torch.Generator(device="cuda").manual_seed(3)
    u = torch.randn((lat.V, 4, 3, 3), dtype=torch.complex128, device="cuda", generator=g)
    lat.set_gauge(torch.linalg.qr(u)[0].contiguous())
    op = dwf.Op(lat, Ls, 1.6, 0.05, 1.0, 0.0, 1.0)
    W1, W2 = optc.random_weights(1, 5)
    one, two = dwf.PtcModel(1), dwf.PtcModel(2)
    one.set_weights(W1, W2)
    two.set_weights(np.concatenate([W1, 0 * W1], axis=1), np.concatenate([W2, 0 * W2], axis=2))
    r = torch.randn((Ls, lat.Vh, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    a, b = torch.empty_like(r), torch.empty_like(r)
    one.apply(op, a, r)
    two.apply(op, b, r)
    assert float((a - b).abs().max() / a.abs().max()) < 2e-6


# bricks of whole tiles (24x12x3, 32x8x4), of odd extents (28x14x7) and without a plane of whole tiles (20x20x6)
@pytest.mark.parametrize("dims", [(24, 24, 12, 2), (32, 16, 16, 2), (28, 14, 14, 2), (20, 20, 12, 2)])
def test_brick_orders(dims, monkeypatch):
    """The tables of every brick, and random fields that do not depend on it (a training run on a random system)."""
    import paper_2602_14454_amd as dwf
    step = np.cumprod((1,) + dims[:3])
    lex, nbr = dwf.Lattice(dims).maps()
    assert np.array_equal(np.sort(lex, axis=None), np.arange(2 * lex.shape[1]))
    for d in range(8):
        mu, n = d % 4, dims[d % 4]
        c = lex // step[mu] % n
        assert np.array_equal(nbr[:, d], lex + ((c + (1 if d < 4 else -1)) % n - c) * step[mu])
    hist = []
    for limit in (None, "4096"):
        if limit:
            monkeypatch.setenv("DWF_BRICK_SITES", limit)
        lat, op = _make(dims, 2)[:2]
        M = dwf.PtcModel(2)
        hist.append(np.asarray(M.train([dwf.PtcPairs(op, None, [1, 3], seed=5)], 3, seed=3), dtype=float).ravel()[:3])
    assert np.allclose(hist[0], hist[1], rtol=1e-6, atol=0)   # FP32 sums in another order


# FP64 launches of up to 256 blocks share the directions among the waves (Ls <= 4: four ways, <= 8: two ways)
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((6, 6, 2, 2), 4), ((8, 8, 8, 16), 4), ((8, 8, 8, 18), 3),
                                     ((2, 2, 2, 2), 5), ((6, 2, 6, 2), 7), ((8, 8, 8, 16), 8), ((8, 8, 8, 18), 6)])
@pytest.mark.parametrize("b,c", [(1.0, 0.0), (1.5, 0.5)])
def test_hop_shared_directions(dims, Ls, b, c):
    """The small-lattice hop on both sides of the limits at which its waves share the directions."""
    test_hop_forms_by_lattice_size(dims, Ls, b, c)


def test_noalloc_limit_is_where_it_was():
    """8x8x14x26 with Ls = 15 in FP64: over the limit, which counts an odd multiple of 32 sites per parity; Ls = 14 is not."""
    import torch

    import paper_2602_14454_amd as dwf
    dims = (8, 8, 14, 26)
    lat, op = _make(dims, 15)[:2]
    x = torch.zeros((15, lat.Vh, 4, 3), dtype=torch.complex128, device="cuda")
    with pytest.raises(dwf.DwfError) as e:
        op.apply_normal_noalloc(torch.empty_like(x), x, prec=0)
    assert e.value.status == -2
    op = _make(dims, 14)[1]
    x = torch.zeros((14, lat.Vh, 4, 3), dtype=torch.complex128, device="cuda")
    out = torch.ones_like(x)
    op.apply_normal_noalloc(out, x, prec=0)
    torch.cuda.synchronize()
    assert not out.any()


# 16 sites (part of a block of 64), 64, 96 and 288 (remainders); extents of 2, 6 and 10
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 4, 2), (2, 6, 2, 4), (2, 6, 6, 4), (10, 2, 4, 2)])
def test_plaquette_blocks(dims):
    """Every plane of the plaquette sum around its blocks; tolerance of test_gpu_gauge.py."""
    import paper_2602_14454_amd as dwf
    from oracle import gauge as G
    U = dwfgen.random_su3_links(dims, 0.5, 5)
    assert abs(dwf.gauge_plaquette(_dev(U), dims) - G.plaquette(U, dims)) < 1e-12
