"""GPU parity on 3D grids whose strided axes go in one pass, over plane shapes
with each pair of passes per axis, planes of every size class, and the grids
just beyond the rule: FS steps, the spectral energy and the adjoint.
Tolerances as for the tiled 2D grids."""

import numpy as np
import pytest

from oracle import adjoint as oadj
from oracle import energy as oen
from paper_2306_04322_amd import inputs as I
from parity_util import DISTINCT, announce, fp32_rounded, gpu_or_fail, max_rel, rel_l2

pytestmark = pytest.mark.gpu

# (nx, ny, nz), p
SHAPES = [((8, 8, 8), 8), ((16, 8, 16), 1), ((8, 16, 8), 3), ((32, 32, 16), 4), ((64, 16, 64), 2), ((8, 8, 128), 5),
          ((16, 128, 8), 2), ((8, 32, 64), 4), ((128, 64, 32), 1), ((256, 64, 32), 1), ((8, 256, 8), 3),
          ((8, 16, 256), 1), ((16, 8, 512), 2), ((8, 512, 8), 1), ((64, 64, 64), 4), ((64, 64, 64), 5),
          ((1024, 8, 16), 1), ((16, 128, 32), 7)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,p", SHAPES)
def test_one_pass_strided_axes(n, p, prec):
    torch = gpu_or_fail()
    from paper_2306_04322_amd.pfspec import Solver
    cfg = I.make_config(3, n, (1.0, 0.9, 1.1), p, I.PAPER_FE, **DISTINCT)
    u0 = I.random_ic(cfg, seed=41)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape(p, 1, 1, 1) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    announce("one-pass strided axes", n, p, prec)
    s = Solver(cfg, prec)
    s.set_fields(u0)
    e, ref = s.energy("fs"), oen.energy(u0, cfg, "fs")
    tol = 1e-12 if prec == "f64" else 2e-6
    for i in range(5):
        assert abs(e[i] - ref[i]) <= tol * max(abs(ref[i]), 1e-3 * abs(ref[0])), (i, e, ref)
    s.step_fs(0.01, 2)
    s.step_fs(0.01, 1)
    traj = oadj.trajectory(u0, cfg, 0.01, 3)
    errs = rel_l2(s.get_fields(), traj[-1])
    assert max_rel(errs) <= (1e-11 if prec == "f64" else 2e-5), errs
    if np.prod(n) > 100000:
        return
    w = I.random_direction(cfg, 42)
    lam = torch.as_tensor(w).to(s.device, s.dtype).contiguous()
    ck = torch.as_tensor(u0).to(s.device, s.dtype).contiguous()
    dpar = s.adjoint_fs(0.01, 3, ck, lam, s.segment_store(3), np.zeros(4))
    rlam, rpar = oadj.fs_adjoint(traj, w, cfg, 0.01)
    err = np.linalg.norm(lam.double().cpu().numpy() - rlam) / np.linalg.norm(rlam)
    perr = np.max(np.abs(dpar - rpar) / np.maximum(np.abs(rpar), 1e-12 * np.max(np.abs(rpar))))
    print("lambda", err, "parameters", perr)
    assert err <= (1e-10 if prec == "f64" else 1e-4)
    # (FP64 only: for these directions dJ/dM cancels to 1e-4 of its terms, and
    # the rounding of FP32 fields alone is 1e-3 of what is left)
    if prec == "f64":
        assert perr <= 1e-9
