"""The far field through cell moments, at sizes past its dispatch rule (24
million pairs; 36 million for the modes with h), against the assembled
matrices, the oracle's sums, and itself with the nodes dealt to other cells."""
import warnings

import numpy as np
import pytest
import torch

from synth.geometry import (Curve, Geometry, clustered_ellipse, clustered_flat_surface, ellipse,
                            fourier_surface, graph_bottom, trig_potential)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def ww():
    from paper_2108_01786_amd import wwbi
    warnings.simplefilter("ignore", RuntimeWarning)
    return wwbi


@pytest.fixture(scope="module")
def ctx(ww):
    c = ww.Context(0)
    yield c
    c.close()


def cell(M0, M1, Mo, seed=0):
    rng = np.random.default_rng(seed)
    c = 0.01 * np.exp(-np.arange(2, 8) / 3.0) * (rng.standard_normal(6) + 1j * rng.standard_normal(6))
    curves = [fourier_surface(M0, 0.08, c), graph_bottom(M1, -1.1, [(1, 0.05)])]
    q = min(0.22, 2.0 / max(1, len(Mo)))
    centres = [(2 * j + 1) * np.pi / max(1, len(Mo)) - 0.5j for j in range(len(Mo))]
    curves += [ellipse(m, z.real, z.imag, q, 0.14, 0.0) for m, z in zip(Mo, centres)]
    return Geometry(curves, np.array(centres), rng.uniform(-1, 1, len(Mo)), 1.0)


def near(gap):
    return Geometry([clustered_flat_surface(4096, np.pi, 0.9), graph_bottom(258, -1.0),
                     clustered_ellipse(2050, np.pi, -gap - 0.15, 0.3, 0.15, 1.5 * np.pi, 0.9)],
                    np.array([np.pi - (gap + 0.15) * 1j]), np.array([0.5]), 1.0)


# cells that straddle boundaries, a last cell that is not full, boundaries of
# less than a cell, whole cells only, and clustered nodes close to each other
GEOMS = {"ragged": lambda: cell(3000, 1502, (754, 754)), "many": lambda: cell(2050, 1026, (258,) * 8),
         "tiny": lambda: cell(4098, 802, (34, 66)), "whole": lambda: cell(4096, 2048, (1024,) * 2),
         "near": lambda: near(0.005)}


@pytest.mark.parametrize("name", GEOMS)
def test_products_match_the_matrix(ww, ctx, name):
    geom = GEOMS[name]()
    n = geom.Mtot
    print(f"case cells product {name} n={n}", flush=True)
    dg = ww.DeviceGeometry.from_synth(geom, DEV)
    A = ctx.debug_matrix(dg)
    x = torch.as_tensor(np.random.default_rng(1).standard_normal(n), device=DEV)
    for T in (False, True):
        y, _ = ctx.matvec(dg, x, mode=ww.MATVEC_ON_THE_FLY, transpose=T)
        ref = (A.T if T else A) @ x
        # a term's error is up to 8 units of rounding of |zeta' kappa|, whose
        # sums are within some 10 times those of its parts
        size = ((A.T if T else A).abs() @ x.abs()).max()
        assert float((y - ref).abs().max()) <= 128 * EPS * float(size), T


def test_normal_velocity_matches_the_matrix(ww, ctx):
    """U = (H gamma_0 / 2 + T gamma) / s of a flow without multi-valued part, T
    (the targets' flavour with h) assembled."""
    geom = cell(6002, 1030, (514,))
    geom = Geometry(geom.curves, geom.zc, 0.0 * geom.a, 0.0)
    print(f"case cells U n={geom.Mtot}", flush=True)
    dg = ww.DeviceGeometry.from_synth(geom, DEV)
    phi = trig_potential(6002, [0.1, 0.05, 0.02], [0.05, 0.0, 0.03])
    U, om, _, _ = ctx.solve_phi(dg, torch.as_tensor(phi, device=DEV), tol=1e-14)
    parts = [ctx.spectral(w.contiguous(), ww.OP_D) for w in torch.split(om, geom.M)]
    gam = torch.cat([-parts[0]] + parts[1:])
    hg = ctx.spectral(gam[:6002].contiguous(), ww.OP_H)
    T = ctx.debug_matrix(dg, which=ww.MAT_T)
    s = torch.as_tensor(np.abs(geom.curves[0].d), device=DEV)
    ref = (0.5 * hg + T @ gam) / s
    # as above, for T, H and D's row sums; T + h and h each below 10 times T
    size = ((T.abs() @ gam.abs()).max() + hg.abs().max()) / s.min()
    assert float((U - ref).abs().max()) <= 256 * EPS * float(size)


def test_other_cells_same_result(ww, ctx):
    """Every boundary's nodes renumbered from another start: the sums are the
    same, over other cells (the pressure takes the stream function's and both
    F operators); and the wall and gamma_t systems against their stored
    matrices."""
    geom = cell(6002, 4098, (1030, 1030))
    print(f"case cells renumbered n={geom.Mtot}", flush=True)
    shift = (17, 33, 5, 50)
    roll = [Curve(np.roll(c.z, -s), np.roll(c.d, -s), np.roll(c.e, -s))
            for c, s in zip(geom.curves, shift)]
    geom2 = Geometry(roll, geom.zc, geom.a, geom.V1)
    phi = trig_potential(6002, [0.1, 0.05], [0.05, 0.03])
    V = trig_potential(6002, [0.1, 0.05], [0.0, 0.1])
    g0 = trig_potential(6002, [0.2, 0.1], [0.1, -0.1])
    kw = dict(tol=1e-14, check=False)
    # dphi/ds and the energy (sources' and targets' flavours with h) of one
    # omega: sums of the same terms over other cells
    dg, dg2 = (ww.DeviceGeometry.from_synth(g, DEV) for g in (geom, geom2))
    _, om, _, _ = ctx.solve_phi(dg, torch.as_tensor(phi, device=DEV), **kw)
    om2 = torch.cat([torch.roll(a, -s) for a, s in zip(torch.split(om, geom.M), shift)])
    d1, E1, _ = ctx.tangential_energy(dg, om, torch.as_tensor(phi, device=DEV), tau=0.1)
    d2, E2, _ = ctx.tangential_energy(dg2, om2, torch.as_tensor(np.roll(phi, -17), device=DEV), tau=0.1)
    d2 = torch.cat([torch.roll(a, s) for a, s in zip(torch.split(d2, geom.M), shift)])
    assert float((d2 - d1).abs().max()) <= 1e-11 * float(d1.abs().max())
    assert abs(E2 - E1) <= 1e-12 * abs(E1)
    z = torch.as_tensor([0.3 - 0.2j, 1.0 - 0.9j, 3.0 - 0.3j], device=DEV)
    out = []
    for g, s in ((geom, 0), (geom2, 17)):
        dg = ww.DeviceGeometry.from_synth(g, DEV)
        p, v, w = (torch.as_tensor(np.roll(a, -s), device=DEV) for a in (phi, V, g0))
        pr, _ = ctx.pressure(dg, p, z, tau=0.1, **kw)
        Ug, gw, _ = ctx.solve_gamma(dg, w, **kw)
        if s == 0:
            st = dict(kw, matvec=ww.MATVEC_STORED)
            gt, _, _, _ = ctx.solve_gamma_t(dg, p, v, tau=0.1, **kw)
            gts, _, _, _ = ctx.solve_gamma_t(dg, p, v, tau=0.1, **st)
            Us, gs, _ = ctx.solve_gamma(dg, w, **st)
            assert float((gt - gts).abs().max()) <= 1e-9 * float(gts.abs().max())
            assert float((gw - gs).abs().max()) <= 1e-11 * float(gs.abs().max())
            assert float((Ug - Us).abs().max()) <= 1e-11 * float(Us.abs().max())
        out.append((pr.cpu(), Ug.cpu(), gw.cpu()))
    (pr, U, gw), (pr2, U2, gw2) = out
    # U, a derivative of the densities, carries up to 2e-11 on such grids
    assert float((pr2 - pr).abs().max()) <= 1e-10 * float(pr.abs().max())
    assert float((torch.roll(U2, 17) - U).abs().max()) <= 1e-11 * float(U.abs().max())
    backw = torch.cat([torch.roll(b, s) for b, s in zip(torch.split(gw2, geom.M[1:]), shift[1:])])
    assert float((backw - gw).abs().max()) <= 1e-11 * float(gw.abs().max())
