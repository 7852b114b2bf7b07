"""GPU parity of the row pass's forms at the edges of the rules that choose
between them (k_row.inc): rows of at most 256 points take one of three forms
by row count, and every order-parameter count has instantiations of its own.

Tolerance: six steps of the seeded state, as for the other shapes of the FS
parity tests (FP64 1e-11, FP32 2e-5 relative L2 per field)."""

import numpy as np
import pytest

from oracle import fs as ofs
from paper_2306_04322_amd import inputs as I
from parity_util import DISTINCT, announce, fp32_rounded, gpu_or_fail, max_rel, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [
    # several rows per wavefront, fewer rows than one work-group holds, odd p
    (2, (8, 8), 1), (2, (8, 64), 3), (2, (16, 8), 5), (2, (32, 16), 6), (2, (64, 8), 7),
    (2, (128, 32), 3), (2, (256, 8), 5), (2, (512, 8), 3), (2, (1024, 8), 7), (2, (2048, 8), 5),
    # 8-point rows: the last row count of the form for few rows, the first of
    # the regular wave form, the first of the register form
    (3, (8, 128, 256), 1), (3, (8, 256, 256), 1), (3, (8, 512, 256), 1),
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ndim,n,p", SHAPES)
def test_row_form_parity(ndim, n, p, prec):
    gpu_or_fail()
    from paper_2306_04322_amd.pfspec import Solver
    cfg = I.make_config(ndim, n, (1.0, 0.9, 1.1)[:ndim], p, I.PAPER_FE, **DISTINCT)
    u0 = I.random_ic(cfg, seed=17)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape((p,) + (1,) * ndim) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    steps = 6 if np.prod(n) < 100000 else 2
    announce("row forms", ndim, n, p, prec)
    s = Solver(cfg, prec)
    s.set_fields(u0)
    s.step_fs(0.01, steps - 1)
    s.step_fs(0.01, 1)
    errs = rel_l2(s.get_fields(), ofs.fs_run(u0, cfg, 0.01, steps))
    assert max_rel(errs) <= (1e-11 if prec == "f64" else 2e-5), errs


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ndim,n,p", [(2, (8, 8), 1), (2, (32, 16), 3), (2, (256, 8), 5), (2, (512, 16), 7),
                                      (3, (8, 128, 256), 1), (3, (8, 256, 256), 1)])
def test_adjoint_row_form_parity(ndim, n, p, prec):
    """The adjoint row pass's forms, two segments of two steps (the parameter
    sums run over the steps of a segment); tolerances as in the adjoint's
    other parity tests."""
    torch = gpu_or_fail()
    from oracle import adjoint as oadj
    from paper_2306_04322_amd.pfspec import Solver
    cfg = I.make_config(ndim, n, (1.0, 0.9, 1.1)[:ndim], p, I.PAPER_FE, **DISTINCT)
    u0 = I.random_ic(cfg, seed=18)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape((p,) + (1,) * ndim) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    w = I.random_direction(cfg, 19)
    announce("adjoint row forms", ndim, n, p, prec)
    s = Solver(cfg, prec)
    s.set_fields(u0)
    ck = [s.fields.clone()]
    s.step_fs(0.01, 2)
    ck.append(s.fields.clone())
    lam = torch.as_tensor(w).to(s.device, s.dtype).contiguous()
    seg = s.segment_store(2)
    dpar = np.zeros(4)
    for c in reversed(ck):
        dpar = s.adjoint_fs(0.01, 2, c, lam, seg, dpar)
    rlam, rpar = oadj.fs_adjoint(oadj.trajectory(u0, cfg, 0.01, 4), w, cfg, 0.01)
    err = np.linalg.norm(lam.double().cpu().numpy() - rlam) / np.linalg.norm(rlam)
    perr = np.max(np.abs(dpar - rpar) / np.maximum(np.abs(rpar), 1e-12 * np.max(np.abs(rpar))))
    print("lambda", err, "parameters", perr)
    assert err <= (1e-10 if prec == "f64" else 1e-4)
    assert perr <= (1e-9 if prec == "f64" else 1e-3)
