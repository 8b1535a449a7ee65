"""GPU kernels chosen by size, width or precision, at the sizes where the choice or the kernel's
edges can go wrong, against the oracle's dense matrix.

Tolerance of the FP64 products: a row sums N products of kernel values and densities, each
within a few units of 1.1e-16 of the oracle's; N <= 4096 of them in any order differ by at most
N x 1.1e-16 x a few = 2e-12 of the largest row in the worst case and by its square root in
practice, so 1e-12 of the largest entry holds with room.
"""
import numpy as np
import pytest

import oracle
from lspr_inputs import merge_surfaces, octasphere, perturbed_ellipsoid, place_at_gap

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_1812_10722_amd import lspr
    assert torch.cuda.is_available()
    return lspr


def _surfaces(nu, nu_blobs=()):
    out = [octasphere(nu, 8.0)]
    rng = np.random.default_rng(nu)
    for k, nb in enumerate(nu_blobs):
        bv, bt = perturbed_ellipsoid(nb, (1.5, 4.0, 1.5), rng)
        out.append((place_at_gap(bv, [0.1, 0.2, 1.0 - 2.0 * k], 8.0, 0.8), bt))
    return out


def _system(surfs, ncol, seed, **rules):
    """x, permittivities and the oracle's products for ncol columns."""
    v, t, sid = merge_surfaces(surfs)
    V, K = oracle.dense_operators(v, t, **rules)
    normal = oracle.panel_geometry(v, t)["normal"]
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((ncol, 2 * len(t))) + 1j * rng.standard_normal((ncol, 2 * len(t)))
    em = 1.7 + 0.05 * rng.random(ncol) + 0.01j * rng.random(ncol)
    es = np.concatenate([(-3.0 + rng.random((ncol, 1)) + 0.3j),
                         2.0 + rng.random((ncol, len(surfs) - 1)) + 0.1j], 1)
    ref = np.stack([oracle.assemble_system(V, K, sid, normal, em[c], es[c], [0, 0, 1.0])[0] @ x[c]
                    for c in range(ncol)])
    return x, em, es, ref


def _worst(y, ref):
    return (np.abs(y - ref).max(1) / np.abs(ref).max(1)).max()


# direct FP64 sums on the fly (one and two wavelengths; every far rule): 8 panels (one partial
# chunk, fewer panels than waves), 288 (a tile past 16 x 16 panels), 968 (ragged chunks), and two
# and three surfaces (own-surface sums apart, ranges that do not start at a tile)
@pytest.mark.parametrize("nu,blobs,ncol,k_far", [(1, (), 1, 4), (6, (), 2, 4), (11, (), 1, 4),
                                                 (5, (3,), 1, 4), (6, (3, 4), 2, 4),
                                                 (5, (3,), 2, 1), (5, (3,), 1, 3), (5, (3,), 2, 7)])
def test_direct_sums_on_the_fly(lib, nu, blobs, ncol, k_far):
    surfs = _surfaces(nu, blobs)
    x, em, es, ref = _system(surfs, ncol, 3, k_far=k_far)
    geo = lib.Geometry(surfs, method="dense", precision="fp64", k_far=k_far, matrix_cores=False)
    y = geo.apply(torch.as_tensor(x).cuda(), em, es).cpu().numpy()
    assert _worst(y, ref) < 1e-12
    again = geo.apply(torch.as_tensor(x).cuda(), em, es, noalloc=True).cpu().numpy()
    assert (again == y).all()


# the same sums with more chunks than CUs: chunks in pairs (an odd one over, pairs across surfaces whose
# ranges differ) against rows of the oracle
@pytest.mark.parametrize("nu,blobs", [(47, ()), (46, (5, 4))])
def test_direct_sums_of_chunk_pairs(lib, nu, blobs):
    surfs = _surfaces(nu, blobs)
    v, t, sid = merge_surfaces(surfs)
    n = len(t)
    rows = np.unique(np.r_[0:5, np.linspace(0, n - 1, 23).astype(int), n - 180:n:20, n - 1])
    V, K = oracle.operators.operator_rows(v, t, rows, 4, 19, 9, 0.5)
    rng = np.random.default_rng(nu)
    x = rng.standard_normal((1, 2 * n)) + 1j * rng.standard_normal((1, 2 * n))
    em, es = np.array([1.7733]), np.array([[-3.38 + 0.2j] + [2.5] * len(blobs)])
    geo = lib.Geometry(surfs, method="dense", precision="fp64", matrix_cores=False)
    y = geo.apply(torch.as_tensor(x).cuda(), em, es).cpu().numpy()[0]
    phi, sig = x[0, :n], x[0, n:]
    same = sid[rows][:, None] == sid[None, :]
    top = 0.5 * phi[rows] + np.where(same, K, 0) @ phi - np.where(same, V, 0) @ sig
    low = 0.5 * phi[rows] - K @ phi + (V * (es[0][sid] / em[0])[None, :]) @ sig
    for got, ref in ((y[rows], top), (y[n + rows], low)):
        assert np.abs(got - ref).max() / np.abs(y).max() < 2e-12  # (17672 products per sum)


# FP32 products of more than 16 wavelengths in half tiles: every number of column groups (3 .. 8),
# each number of waves per group, odd and even K-steps per tile (P = 6, 8, 10, 15) and direct
# tiles of one step (short remainders).  The arithmetic per output is that of the four-wave
# workgroups, so the results are equal bit for bit, on every repeat (a request that had not
# landed would show here).
@pytest.mark.parametrize("p", [6, 8, 10, 12, 15])
def test_half_tile_products_equal_four_wave_products(lib, p):
    surfs = _surfaces(13, (5, 6))
    n = sum(len(t) for _, t in surfs)
    kw = dict(method="treecode", precision="fp32", p=p, theta=0.5)
    four, half = lib.Geometry(surfs, four_wave=True, **kw), lib.Geometry(surfs, **kw)
    rng = np.random.default_rng(p)
    for nl in (17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 57, 64):
        x = torch.as_tensor(rng.standard_normal((nl, 2 * n)) +
                            1j * rng.standard_normal((nl, 2 * n))).cuda()
        em = np.full(nl, 1.7733)
        es = np.stack([-3.0 + 0.3j + rng.standard_normal(nl)] + [np.full(nl, 2.5)] * 2, 1)
        want = four.apply(x, em, es)
        for _ in range(4):
            assert torch.equal(half.apply(x, em, es), want), (p, nl)


# FP64 products of 9 to 32 wavelengths in half tiles: two to four column groups at every order that has
# them, odd and even halves, direct tiles of one step and three surfaces; the same products in the same
# order as the four-wave workgroups, so equal bit for bit, on every repeat
@pytest.mark.parametrize("p", [6, 8, 12, 15])
def test_half_tile_fp64_products_equal_four_wave_products(lib, p):
    surfs = _surfaces(13, (5, 6))
    n = sum(len(t) for _, t in surfs)
    kw = dict(method="treecode", precision="fp64", p=p, theta=0.5)
    four, half = lib.Geometry(surfs, four_wave=True, **kw), lib.Geometry(surfs, **kw)
    rng = np.random.default_rng(p)
    for nl in (9, 13, 16, 17, 24, 25, 32):
        x = torch.as_tensor(rng.standard_normal((nl, 2 * n)) + 1j * rng.standard_normal((nl, 2 * n))).cuda()
        em = np.full(nl, 1.7733)
        es = np.stack([-3.0 + 0.3j + rng.standard_normal(nl)] + [np.full(nl, 2.5)] * 2, 1)
        want = four.apply(x, em, es)
        for _ in range(4):
            assert torch.equal(half.apply(x, em, es), want), nl


# a mesh of few chunks, whose far field is cut into pieces of a few tiles: every launch class (1-16,
# 17-32 and 33-64 wavelengths), several surfaces (own-surface pieces apart) and a ragged last
# chunk; FP32 sums of whole tiles round as before, so 2e-6 of the largest entry bounds them (single
# precision values and densities, 928 of them)
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-6)])
def test_products_of_few_chunks(lib, precision, tol):
    surfs = _surfaces(10, (4,))
    geo = lib.Geometry(surfs, method="dense", precision=precision)
    for ncol in (1, 3, 16, 17, 33, 64):
        x, em, es, ref = _system(surfs, ncol, ncol) if ncol <= 17 else (x, em, es, ref)
        rep = -(-ncol // len(x))
        xs, ems, ess = np.tile(x, (rep, 1))[:ncol], np.tile(em, rep)[:ncol], np.tile(es, (rep, 1))[:ncol]
        want = np.tile(ref, (rep, 1))[:ncol]
        xt = torch.as_tensor(xs).cuda()
        y = geo.apply(xt, ems, ess).cpu().numpy()
        assert _worst(y, want) < tol, ncol
        assert (geo.apply(xt, ems, ess, noalloc=True).cpu().numpy() == y).all()


# products read x and write y in the caller's panel order, also where y is x; permittivities go as a
# kernel argument up to 128 values and by a copy above (64 columns x 3 surfaces)
@pytest.mark.parametrize("noalloc", [False, True])
def test_product_in_place_and_many_permittivities(lib, noalloc):
    surfs = _surfaces(6, (3, 4))
    x, em, es, ref = _system(surfs, 8, 21)
    x, em, es, ref = (np.tile(a, (8,) + (1,) * (a.ndim - 1)) for a in (x, em, es, ref))
    geo = lib.Geometry(surfs, method="dense", precision="fp64")
    for n in (3, 64):
        xt = torch.as_tensor(x[:n]).cuda()
        y = geo.apply(xt, em[:n], es[:n], noalloc=noalloc)
        assert _worst(y.cpu().numpy(), ref[:n]) < 1e-12
        geo.apply(xt, em[:n], es[:n], out=xt, noalloc=noalloc)
        assert torch.equal(xt, y)


# the search for near-singular panels: leaves of one panel (more leaves than one round of a
# workgroup tries) and the default's, and reaches at which targets have a few, dozens (more than a
# wave holds from its counting) and over 64 near panels (a filling pass); small meshes beside a
# sphere, so that chunks hold panels of several shapes and sizes
@pytest.mark.parametrize("nu,threshold,ncrit", [(1, 0.5, 0), (13, 0.5, 1), (13, 0.2, 1), (9, 0.2, 0), (9, 0.1, 3)])
def test_near_panels_of_every_target(lib, nu, threshold, ncrit):
    surfs = _surfaces(nu, (2, 3) if nu > 1 else ())
    x, em, es, ref = _system(surfs, 1, 5, threshold=threshold)
    geo = lib.Geometry(surfs, method="dense", precision="fp64", threshold=threshold, ncrit=ncrit)
    y = geo.apply(torch.as_tensor(x).cuda(), em, es).cpu().numpy()
    assert _worst(y, ref) < 1e-12


# the same search by a walk down the trees for each target (more leaves than trying each for each chunk
# is worth: here one panel per leaf), with few, dozens and over 64 near panels per target, two meshes
# beside the sphere; rows of the oracle
@pytest.mark.parametrize("threshold", [0.5, 0.2, 0.1])
def test_near_panels_by_tree_walk(lib, threshold):
    surfs = _surfaces(29, (6, 5))
    v, t, sid = merge_surfaces(surfs)
    n = len(t)
    rows = np.unique(np.r_[0:n:401, n - 350:n:25, n - 1])
    V, K = oracle.operators.operator_rows(v, t, rows, 4, 19, 9, threshold)
    rng = np.random.default_rng(29)
    x = rng.standard_normal((1, 2 * n)) + 1j * rng.standard_normal((1, 2 * n))
    em, es = np.array([1.7733]), np.array([[-3.38 + 0.2j, 2.5, 2.4]])
    geo = lib.Geometry(surfs, method="dense", precision="fp64", threshold=threshold, ncrit=1)
    y = geo.apply(torch.as_tensor(x).cuda(), em, es).cpu().numpy()[0]
    phi, sig = x[0, :n], x[0, n:]
    same = sid[rows][:, None] == sid[None, :]
    top = 0.5 * phi[rows] + np.where(same, K, 0) @ phi - np.where(same, V, 0) @ sig
    low = 0.5 * phi[rows] - K @ phi + (V * (es[0][sid] / em[0])[None, :]) @ sig
    for got, ref in ((y[rows], top), (y[n + rows], low)):
        assert np.abs(got - ref).max() / np.abs(y).max() < 2e-12  # (7500 products per sum)


# the right-hand side's columns run through V alone: one and two column groups per operator (3, 6 and
# 18 columns) and both precisions, at orders whose narrow products have their own kernels; with
# theta 0.05 every pair is summed directly (tolerances as above), with 0.5 the expansions' relative
# truncation, theta^(p + 1), bounds the error
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-6)])
@pytest.mark.parametrize("p", [6, 8, 15])
@pytest.mark.parametrize("blobs", [(), (4,), (3, 4, 3, 4, 3)])
def test_right_hand_side_through_v_alone(lib, precision, tol, p, blobs):
    surfs = _surfaces(10, blobs)
    v, t, sid = merge_surfaces(surfs)
    V, K = oracle.dense_operators(v, t)
    em, es = 1.7733, np.array([-3.38 + 0.2j] + [2.5] * len(blobs))
    e = np.array([0.3, -0.5, 1.2])
    _, ref = oracle.assemble_system(V, K, sid, oracle.panel_geometry(v, t)["normal"], em, es, e)
    for theta, bound in ((0.05, tol), (0.5, max(tol, 0.5 ** (p + 1)))):
        geo = lib.Geometry(surfs, method="treecode", precision=precision, p=p, theta=theta)
        b = geo.rhs(np.array([em]), es[None], e).cpu().numpy()[0]
        assert np.abs(b - ref).max() / np.abs(ref).max() < bound, theta


# tiles against the same far field evaluated on the fly by kernels of their own, for every order that
# has both (tiles of one and of several slices) and every far rule; both in FP64, where (p + 1)^2 terms of
# products of rounded powers and folded moments stay below 1e-11 of the largest entry
@pytest.mark.parametrize("p,k_far", [(2, 4), (4, 1), (6, 3), (8, 4), (8, 7), (10, 4)])
def test_tiles_equal_sums_on_the_fly(lib, p, k_far):
    surfs = _surfaces(14, (5, 6))
    n = sum(len(t) for _, t in surfs)
    kw = dict(method="treecode", precision="fp64", p=p, theta=0.5, k_far=k_far, ncrit=10, m2p_min_panels=1)
    tiles, fly = lib.Geometry(surfs, **kw), lib.Geometry(surfs, matrix_cores=False, **kw)
    rng = np.random.default_rng(p)
    x = torch.as_tensor(rng.standard_normal((3, 2 * n)) + 1j * rng.standard_normal((3, 2 * n))).cuda()
    em, es = np.full(3, 1.7733), np.tile([-3.0 + 0.3j, 2.5, 2.0 + 0.1j], (3, 1))
    a, b = tiles.apply(x, em, es).cpu().numpy(), fly.apply(x, em, es).cpu().numpy()
    assert _worst(a, b) < 1e-11
