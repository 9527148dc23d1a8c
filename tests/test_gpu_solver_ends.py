"""How a solve ends: on input that makes the system singular or not finite, on
cells that need more steps than a short restart cycle holds, on a small budget
of steps, and when a launch gives up."""
import os
import threading
import time
import warnings

import numpy as np
import pytest
import torch

import oracle as O
from synth.geometry import Geometry, ellipse, fourier_surface, graph_bottom, trig_potential

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


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


def cell(M0, M1, Mo=(), gap=0.35, seed=0):
    """Surface, bottom and a row of ellipses whose tops lie `gap` below y = 0."""
    rng = np.random.default_rng(seed)
    c = 0.01 * np.exp(-np.arange(2, 8) / 3.0) * (rng.standard_normal(6) + 1j * rng.standard_normal(6))
    curves = [fourier_surface(M0, 0.08, c), graph_bottom(M1, -1.1, [(1, 0.05)])]
    q = min(0.22, 2.0 / max(1, len(Mo)))
    centres = [(2 * j + 1) * np.pi / max(1, len(Mo)) - 1j * (gap + 0.14) for j in range(len(Mo))]
    curves += [ellipse(m, z.real, z.imag, q, 0.14, 0.0) for m, z in zip(Mo, centres)]
    geom = Geometry(curves, np.array(centres), rng.uniform(-1, 1, len(Mo)), 1.0)
    return geom, trig_potential(M0, 0.1 * rng.standard_normal(3), 0.1 * rng.standard_normal(3))


def rel(a, b):
    a, b = (np.asarray(v.cpu() if torch.is_tensor(v) else v) for v in (a, b))
    return float(np.abs(a - b).max() / np.abs(b).max())


def options(ww, prec, **kw):
    return dict(precision=ww.FP64 if prec == "fp64" else ww.FP32_REFINED, check=False, **kw)


# one-launch solves, the two-grid iteration's sizes, and the stored matrix
@pytest.mark.parametrize("M0,M1,Mo", [(96, 64, (64,)), (1024, 256, (256,))])
@pytest.mark.parametrize("prec", ["fp64", "refined"])
@pytest.mark.parametrize("mode", ["auto", "stored"])
def test_not_finite_is_no_solution(ww, ctx, M0, M1, Mo, prec, mode):
    """zeta' = 0 at one wall node passes the input checks (finite samples, the
    right orientation) and makes the diagonal's limit 0 / 0."""
    geom, phi = cell(M0, M1, Mo)
    print(f"case zero derivative n={geom.Mtot} {prec} {mode}", flush=True)
    dg0 = ww.DeviceGeometry.from_synth(geom, DEV)
    p = torch.as_tensor(phi, device=DEV)
    kw = options(ww, prec, matvec=ww.MATVEC_AUTO if mode == "auto" else ww.MATVEC_STORED)
    _, omega, _, _ = ctx.solve_phi(dg0, p, **kw)
    geom.curves[2].d[5] = 0.0
    dg = ww.DeviceGeometry.from_synth(geom, DEV)
    bad = (ww.STAGNATED,) if prec == "fp64" else (ww.REFINE_STALLED,)
    ones = torch.ones(M0, dtype=torch.float64, device=DEV)
    assert ctx.solve_phi(dg, p, **kw)[3].status in bad
    assert ctx.solve_gamma(dg, p, **kw)[2].status in bad
    assert ctx.adjoint_phi(dg, omega, ones, **kw)[1].status in bad
    rhs = torch.as_tensor(np.random.default_rng(3).standard_normal((3, geom.Mtot)), device=DEV)
    assert ctx.solve_phi_multi(dg, rhs, **kw)[1].status in bad
    z = torch.as_tensor([0.3 - 0.2j, 1.0 - 0.9j], device=DEV)
    assert ctx.pressure(dg, p, z, tau=0.1, **kw)[1].status in bad
    # the context is as good as before
    _, again, _, r = ctx.solve_phi(dg0, p, **kw)
    assert r.status in (ww.OK, ww.WARN_UNDERRESOLVED) and torch.equal(again, omega)
