"""Kernel variants chosen by size: each at the edges of its range."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _handle(p, **opt):
    from paper_1602_03641_amd import vag
    opt.setdefault("max_iter", 20000)
    opt.setdefault("cfl", p.cfl)
    h = vag.Handle(p, **opt)
    return h, h.solve_pressure()


@pytest.mark.parametrize("dims,B", [((9, 7, 6), 2), ((9, 7, 6), 129), ((13, 4, 3), 64), ((12, 11, 9), 512),
                                    ((12, 11, 9), 900), ((12, 11, 9), 2048)])
def test_ilu_substitutions(dims, B):
    """Block sizes on both sides of what fits in LDS, last blocks ragged,
    levels of more rows than a wavefront takes at once: z = M^-1 r element by
    element against the oracle's block-Jacobi ILU(0) of its own system.  Each
    entry of z is a sum of about 10^2 terms per block row, so 1e-11 of max |z|
    leaves 10^3 over the rounding of the substitutions."""
    from paper_1602_03641_amd import vag
    from oracle import ilu
    p = synth.random_problem(dims, 21, n_patches=4, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, rtol=1e-8, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, ilu_block_rows=B,
                      eliminate_frac_faces=0)
    A, _ = oracle.system(p)
    rows = ilu.bj_ilu0(A, B)
    r = np.random.default_rng(22).standard_normal(A.shape[0])
    z, zr = h.apply_preconditioner(r), ilu.bj_ilu0_apply(rows, r)
    assert np.abs(z - zr).max() <= 1e-11 * np.abs(zr).max()
    h.close()
