"""The 3D kernels (a site's populations spread over the waves of a block) against the FP64 oracle, to the bounds that the other step kernels keep: double 1e-12 on the populations and fields; float
storage (16 + 4 k) 2^-24 on the fields after k steps, and (32 + sqrt k) 2^-24 where the update is in double.

The extents cover runs of 64 sites that end inside a row, hold a row boundary, end a slab of eight rows
early or fill it exactly, rows shorter than a run (down to one site), and patches cut off in y and z.
"""
import math

import pytest
import torch

import workloads as W
from oracle import lattice as OL
from oracle import quadrature as qd

pytestmark = pytest.mark.gpu

STEPS = 2
EXTENTS = [(64, 8, 8), (65, 9, 3), (97, 13, 9), (127, 1, 2), (128, 3, 1), (200, 10, 2), (63, 5, 4), (31, 17, 3),
           (9, 3, 10), (2, 2, 2), (1, 1, 1), (1, 70, 1)]


def check(extent, storage, order=3, bc=None, zeta=1.0, tau=0.8, force=None, quad=None, **kw):
    from paper_1909_04502_amd import rlbm as R
    quad = qd.product_3d(zeta, order) if quad is None else quad
    n, T, u = (torch.tensor(a) for a in W.taylor_green_3d(*extent, 0.1, density_sigma=1e-2, seed=5))
    field = isinstance(tau, torch.Tensor)
    gl = R.Lattice(d=3, zeta=zeta, order=order, extent=extent, storage=storage, tau=0.8 if field else tau,
                   tau_field=tau if field else None, bc=bc, force=force, **kw)
    ol = OL.Lattice(quad, tau, extent, bc=bc, force=force, tau_T=kw.get("tau_T", 0.0))
    f0, first = gl.init(n, T, u, want_fields=True)
    res, last = gl.step(f0, gl.new_state(), STEPS, want_last=True)
    now = gl.moments(res)
    gl.sync()
    init = ol.init(n, T, u)
    fs = ol.collide(init)
    for _ in range(STEPS):
        pre = ol.stream(fs)
        fs = ol.collide(pre)
    ref = ol.macro(pre)
    tol = {"f64": 1e-12, "f32dev": (16 + 4 * STEPS) * 2.0 ** -24, "f32dev_f64": (32 + math.sqrt(STEPS)) * 2.0 ** -24}[storage]
    refs = [(first, ol.macro(init)), (last, ref), (now, ol.macro(ol.stream(fs)))]
    pairs = [(got[k].cpu(), want[k]) for got, want in refs for k in ("n", "eps", "T", "U")]
    if storage == "f64":
        pairs.append((res.cpu(), fs))
    for a, b in pairs:
        assert (a - b).abs().max().item() <= tol * b.abs().max().item()


@pytest.mark.parametrize("extent", EXTENTS)
@pytest.mark.parametrize("storage", ["f64", "f32dev", "f32dev_f64"])
def test_split_step_against_the_oracle(extent, storage):
    print(f"[case] split {extent} {storage}", flush=True)
    check(extent, storage)


@pytest.mark.parametrize("order,zeta", [(2, 1.0), (2, 0.0), (3, 0.0), (3, 4.0)])
@pytest.mark.parametrize("bc", [("open",) * 3, ("open", "periodic", "periodic"), ("periodic", "open", "open")])
def test_split_step_orders_masses_and_boundaries(order, zeta, bc):
    print(f"[case] split order {order} zeta {zeta} {bc}", flush=True)
    check((70, 11, 9), "f64", order, bc, zeta)
    check((20, 11, 9), "f32dev", order, bc, zeta)


def test_split_step_takes_a_tau_field():
    print("[case] split tau field", flush=True)
    check((70, 11, 9), "f64", tau=torch.tensor(W.random_field((9, 11, 70), 3, 0.7, 1.1)))


@pytest.mark.parametrize("storage", ["f64", "f32dev", "f32dev_f64"])
@pytest.mark.parametrize("extent", [(66, 9, 3), (20, 4, 9)])
def test_split_step_force_and_walls(extent, storage):
    print(f"[case] split walls {extent} {storage}", flush=True)
    check(extent, storage, bc=("wall", "periodic", "open"), force=(1e-3, -2e-3, 3e-3))
    check(extent, storage, order=2, bc=("periodic", "wall", "wall"), force=(0.0, 0.0, 1e-3))


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("extent", [(64, 8, 8), (65, 9, 3), (131, 3, 3), (20, 11, 5), (3, 3, 3)])
def test_split_massive_rule(extent, storage):
    print(f"[case] split massive {extent} {storage}", flush=True)
    v0 = 0.2719557997821228
    check(extent, storage, zeta=5.0, quad=qd.massive_onlattice(3, 5.0, 3, v0), kind="massive_onlattice", v0=v0)
    if storage == "f32dev":
        check(extent, storage, zeta=5.0, quad=qd.massive_onlattice(3, 5.0, 3, v0), kind="massive_onlattice", v0=v0,
              bc=("wall", "periodic", "open"), force=(0.0, 1e-3, 0.0))


@pytest.mark.parametrize("storage", ["f64", "f32dev"])
@pytest.mark.parametrize("extent,bc", [((640, 1, 1), ("periodic", "open", "open")), ((65, 7, 6), None),
                                       ((13, 9, 8), ("open", "periodic", "open")), ((6, 6, 6), None)])
def test_split_massless_rule(extent, bc, storage):
    print(f"[case] split massless {extent} {storage}", flush=True)
    check(extent, storage, zeta=0.0, quad=qd.ur_onlattice_3d(3), kind="ur_onlattice", bc=bc, tau=0.6, tau_T=0.3)


@pytest.mark.parametrize("extent,storage", [((20, 41, 43), "f64"), ((67, 43, 41), "f32dev"), ((66, 48, 41), "f64"),
                                            ((3, 130, 129), "f32dev_f64")])
def test_split_step_of_many_patches(extent, storage):
    """36 patches and more, cut off in y and z, in whole patches and in eighths, and 289 of them."""
    print(f"[case] split patches {extent} {storage}", flush=True)
    check(extent, storage, order=2, zeta=0.0)   # (the oracle's equation of state is fast without a mass)


@pytest.mark.parametrize("kind", ["massive_onlattice", "ur_onlattice"])
def test_split_onlattice_of_many_patches(kind):
    print(f"[case] split patches {kind}", flush=True)
    v0 = 0.2719557997821228
    if kind == "massive_onlattice":
        check((5, 41, 43), "f32dev", zeta=5.0, quad=qd.massive_onlattice(3, 5.0, 3, v0), kind=kind, v0=v0)
    else:
        check((9, 41, 43), "f64", zeta=0.0, quad=qd.ur_onlattice_3d(3), kind=kind, tau=0.6, tau_T=0.3)
