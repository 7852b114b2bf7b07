"""GPU parity of the adjoint row pass's forms (k_adj.inc) at the lines between
them: 1024-point float rows of every order-parameter count that has a
work-group of its own, 4096-point float rows on both sides of the count read at
run time, 512-point double rows with eight, and the last row
count of the form for few rows with the first of the regular one.

The loss is half the squared deviation of the fields from their mean, whose
derivative has no cancellation in any parameter.  Tolerances as in the
adjoint's other parity tests (FP64 1e-10 and 1e-9 of each parameter, FP32 1e-4
and 1e-3)."""

import numpy as np
import pytest

from oracle import adjoint as oadj
from paper_2306_04322_amd import inputs as I
from parity_util import DISTINCT, announce, fp32_rounded, gpu_or_fail

pytestmark = pytest.mark.gpu

SHAPES = [(2, (1024, 8), p, "f32") for p in range(1, 9)] + [(2, (1024, 128), 5, "f32")]
SHAPES += [(2, (4096, 8), p, "f32") for p in (2, 3, 7, 8)]
SHAPES += [(2, (512, n), 8, "f64") for n in (8, 64)]
SHAPES += [(2, (256, n), 1, "f64") for n in (512, 1024)] + [(3, (32, 32, 64), 6, "f64"), (3, (8, 128, 256), 2, "f64")]


@pytest.mark.parametrize("ndim,n,p,prec", SHAPES)
def test_adjoint_form(ndim, n, p, prec):
    torch = gpu_or_fail()
    from paper_2306_04322_amd.pfspec import Solver
    cfg = I.make_config(ndim, n, (1.0, 0.9, 1.1)[:ndim], p, I.PAPER_FE, **DISTINCT)
    u0 = I.random_ic(cfg, seed=51)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape((p,) + (1,) * ndim) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    traj = oadj.trajectory(u0, cfg, 0.01, 3)
    w = traj[-1] - traj[-1].mean(axis=tuple(range(1, ndim + 1)), keepdims=True)
    announce("adjoint forms", ndim, n, p, prec)
    s = Solver(cfg, prec)
    lam = torch.as_tensor(w).to(s.device, s.dtype).contiguous()
    ck = torch.as_tensor(u0).to(s.device, s.dtype).contiguous()
    dpar = s.adjoint_fs(0.01, 3, ck, lam, s.segment_store(3), np.zeros(4))
    rlam, rpar = oadj.fs_adjoint(traj, w, cfg, 0.01)
    err = np.linalg.norm(lam.double().cpu().numpy() - rlam) / np.linalg.norm(rlam)
    perr = np.max(np.abs(dpar - rpar) / np.abs(rpar))
    print("lambda", err, "parameters", perr, rpar)
    assert err <= (1e-10 if prec == "f64" else 1e-4)
    assert perr <= (1e-9 if prec == "f64" else 1e-3)


@pytest.mark.parametrize("n,p", [((8, 8, 8), 8), ((8, 16, 8), 3), ((32, 32, 16), 4), ((64, 16, 64), 2), ((8, 32, 64), 5),
                                 ((8, 512, 8), 1), ((16, 128, 32), 7)])
def test_one_pass_axes_parameters_fp32(n, p):
    """The parameter gradients in FP32 on 3D grids whose strided axes go in
    one pass."""
    test_adjoint_form(3, n, p, "f32")
