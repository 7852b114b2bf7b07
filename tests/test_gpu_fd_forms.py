"""GPU parity of the FD step's fused kernels (k_fd.hip) with the oracle, on
grids at the edges of their tiles and of the rule that chooses between them:
2D tiles narrower than a row, one row high, cut off by the grid; 3D tiles of
each shape; marching blocks whose rows and planes do not divide the grid; the
two-kernel step beside them.

Tolerance: as for the FD step's other parity tests (FP64 1e-12, FP32 1e-5
relative L2 per field over 20 steps; here at most 5)."""

import numpy as np
import pytest

from oracle import fd as ofd
from paper_2306_04322_amd import inputs as I
from parity_util import DISTINCT, announce, fp32_rounded, gpu_or_fail, max_rel, rel_l2

pytestmark = pytest.mark.gpu

SMALL = [(2, (8, 8), 1), (2, (16, 8), 3), (2, (64, 16), 5), (2, (512, 8), 8), (2, (4096, 16), 2),
         (2, (8, 1024), 2), (2, (256, 128), 7),
         (3, (8, 8, 8), 1), (3, (16, 8, 16), 8), (3, (32, 16, 8), 3), (3, (64, 8, 32), 5),
         (3, (64, 16, 8), 8), (3, (128, 8, 16), 4), (3, (128, 8, 8), 6), (3, (256, 8, 8), 2)]
# float: the 512- and the 768-lane marching form; double: the latter; and the
# two-kernel step
LARGE = [((256, 256, 64), 4, "f32"), ((512, 128, 128), 3, "f32"), ((128, 128, 256), 2, "f32"),
         ((256, 128, 128), 2, "f64"), ((128, 128, 256), 4, "f64"), ((128, 64, 64), 8, "f64")]


def _check(ndim, n, p, prec, steps):
    gpu_or_fail()
    from paper_2306_04322_amd.pfspec import Solver
    cfg = I.make_config(ndim, n, (1.0, 0.9, 1.1)[:ndim], p, I.PAPER_FE, **DISTINCT)
    u0 = I.random_ic(cfg, seed=21)
    u0[1:] = 0.5 * u0[1:] + 0.3 * np.arange(1, p + 1).reshape((p,) + (1,) * ndim) / p
    if prec == "f32":
        u0 = fp32_rounded(u0)
    announce("fd forms", ndim, n, p, prec)
    s = Solver(cfg, prec)
    s.set_fields(u0)
    s.step_fd(2e-4, steps)
    errs = rel_l2(s.get_fields(), ofd.fd_run(u0, cfg, 2e-4, steps))
    assert max_rel(errs) <= (1e-12 if prec == "f64" else 1e-5), errs


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ndim,n,p", SMALL)
def test_fd_small_forms(ndim, n, p, prec):
    _check(ndim, n, p, prec, 5)


@pytest.mark.parametrize("n,p,prec", LARGE)
def test_fd_large_forms(n, p, prec):
    _check(3, n, p, prec, 2)
