"""GPU parity of the FD step with the oracle on both sides of the 3D
rule's lines (k_fd.hip).

Tolerance: as for the FD step's other parity tests (FP64 1e-12, FP32 1e-5
relative L2 per field over 20 steps; here at most 5)."""

import numpy as np
import pytest

from oracle import fd as ofd
from paper_2306_04322_amd import inputs as I
from parity_util import DISTINCT, announce, fp32_rounded, gpu_or_fail, max_rel, rel_l2

pytestmark = pytest.mark.gpu

# the two-kernel step below the marching form's line, tiles below theirs
LINES = [((64, 128, 256), 5, "f32"), ((128, 256, 128), 4, "f32"), ((32, 256, 128), 1, "f32"), ((32, 128, 128), 1, "f32"),
         ((16, 128, 128), 4, "f64"), ((32, 64, 128), 3, "f64"), ((64, 256, 128), 2, "f64")]


def _check(n, p, prec, fe, dt, steps):
    gpu_or_fail()
    from paper_2306_04322_amd.pfspec import Solver
    ndim = len(n)
    cfg = I.make_config(ndim, n, (1.0, 0.9, 1.1)[:ndim], p, fe, **DISTINCT)
    u0 = I.random_ic(cfg, seed=71)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape((p,) + (1,) * ndim) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    announce("fd lines", fe["kind"], n, p, prec)
    s = Solver(cfg, prec)
    s.set_fields(u0)
    s.step_fd(dt, steps)
    errs = rel_l2(s.get_fields(), ofd.fd_run(u0, cfg, dt, steps))
    assert max_rel(errs) <= (1e-12 if prec == "f64" else 1e-5), errs


@pytest.mark.parametrize("n,p,prec", LINES)
def test_fd_large(n, p, prec):
    _check(n, p, prec, I.PAPER_FE, 2e-4, 2)
