"""The LDS-staged pull at the edges of its 64 x 4 tiles: any x extent, boundary, wall and force, alone and in a batch.

The staged kernels read the same taps with the same weights in the same order as the register kernels (variant 1;
runs of 256 sites in a batch), so the states are equal bit for bit: no tolerance.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

REG, LDS = 1, 12            # register kernel in 64 x 4 band tiles; the staged kernel
BATCH_RUNS, BATCH_LDS = 3, 0
PP = ("periodic", "periodic")


@pytest.mark.parametrize("order,storage,ext,bc,force", [
    (3, "f64", (1, 1), PP, None),
    (3, "f64", (63, 3), PP, None),
    (2, "f64", (65, 5), ("open", "open"), None),
    (3, "f64", (128, 6), ("open", "periodic"), None),   # 16 bytes per lane: whole tiles; a row of one chunk
    (2, "f64", (2, 3), PP, None),
    (3, "f64", (66, 5), ("open", "periodic"), None),
    (3, "f64", (129, 9), ("wall", "periodic"), (0.0, 3e-4)),
    (3, "f32dev", (61, 4), ("periodic", "wall"), (2e-4, 0.0)),
    (2, "f32dev", (127, 6), ("open", "periodic"), None),
    (3, "f32dev", (3, 130), PP, None),
    (3, "f32dev_f64", (193, 7), ("wall", "open"), None),
    (2, "f32dev_f64", (64, 2), PP, None)])
def test_staged_equals_register_kernel_at_tile_edges(order, storage, ext, bc, force):
    from paper_1909_04502_amd import rlbm as R
    print(f"[case] stage {order} {storage} {ext} {bc}", flush=True)
    kw = {"force": force} if force else {}
    gl = R.Lattice(d=2, zeta=1.0, order=order, extent=ext, bc=bc, storage=storage, tau=0.8, **kw)
    n, T, u = (torch.tensor(a) for a in W.taylor_green_2d(*ext, 0.1, density_sigma=1e-3, seed=3))
    f0 = gl.init(n, T, u, torch.tensor(W.population_noise(gl.Q, tuple(reversed(ext)), seed=4)), 1e-3)
    out = []
    for v in (REG, LDS):
        gl.variant = v
        out.append(gl.step(f0.clone(), gl.new_state(), 5).cpu())
        gl.sync()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("storage,ext,bc,staged", [("f64", (725, 725), PP, True), ("f64", (723, 724), PP, False),
                                                   ("f32dev", (1025, 1025), ("open", "periodic"), True)])
def test_default_step_is_staged_past_256_mib(storage, ext, bc, staged):
    """Both sides of the rule (two order-3 states of 257, 256 and 257 MiB): the default equals the register kernel."""
    from paper_1909_04502_amd import rlbm as R
    print(f"[case] stage default {storage} {ext}", flush=True)
    gl = R.Lattice(d=2, zeta=1.0, order=3, extent=ext, bc=bc, storage=storage, tau=0.8)
    assert (2 * gl.Q * gl.sites * (8 if storage == "f64" else 4) > 256 << 20) == staged
    n, T, u = (torch.tensor(a) for a in W.taylor_green_2d(*ext, 0.1, density_sigma=1e-3, seed=3))
    f0 = gl.init(n, T, u)
    a = gl.step(f0.clone(), gl.new_state(), 2)
    gl.variant = REG
    b = gl.step(f0.clone(), gl.new_state(), 2)
    gl.sync()
    assert torch.equal(a, b)


@pytest.mark.parametrize("storage,order", [("f64", 3), ("f64", 2), ("f32dev", 3), ("f32dev_f64", 3)])
@pytest.mark.parametrize("ext", [True, False])
def test_staged_batch_equals_runs_of_sites(storage, order, ext):
    from paper_1909_04502_amd import rlbm as R
    print(f"[case] stage batch {storage} {order} {ext}", flush=True)
    sizes = [(64, 4), (1, 1), (65, 3), (63, 130), (200, 5), (31, 33), (128, 9)]
    specs = [{"extent": e, "tau": 0.7 + 0.1 * i, "zeta": 0.5 * i} for i, e in enumerate(sizes)]
    if ext:
        specs[4].update(bc=("wall", "periodic"), force=(0.0, 2e-4))
    b = R.Batch(specs, order=order, storage=storage)
    f = [[torch.tensor(a) for a in W.taylor_green_2d(*e, 0.05, density_sigma=1e-3, seed=5 + i)]
         for i, e in enumerate(sizes)]
    f0 = b.init(*[[x[k] for x in f] for k in range(3)])
    out = []
    for v in (BATCH_RUNS, BATCH_LDS):
        b.variant = v
        out.append(b.step(f0.clone(), b.new_state(), 5).cpu())
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
