"""The flow's traversal in slabs along z: a thinner last slab, site counts that
are no multiple of a workgroup's 64 sites, an even and an odd number of stages
(the result leaves through the layout kernel or the last stage) and steps so
long that the exponential squares, every link against the FP64 oracle.  The
bound is that of the other flow tests: some 1e3 operations of order one in a
stage, at most nine stages, 1e-16 each."""
import numpy as np
import pytest

from oracle import flow as F
from paper_1701_07559_amd import inputs as I

import test_gpu_flow as TF

pytestmark = pytest.mark.gpu
M = TF.M


@pytest.mark.parametrize("dims,eps,nsteps", [((2, 3, 17, 3), 0.05, 1), ((3, 2, 19, 2), 0.05, 2), ((4, 4, 24, 2), 0.03, 3),
                                             ((2, 2, 2, 2), 0.4, 1), ((16, 2, 9, 2), 0.4, 2)])
def test_flow_slabs(M, dims, eps, nsteps):
    U = I.random_links(dims, 0.5, 95)
    V, (p0, p1) = M.mdwf_wilson_flow(dims, U, eps, nsteps)
    ref = F.flow(U, eps, nsteps)
    assert np.abs(V - ref).max() <= 1e-12
    assert abs(p0 - F.plaquette(U)) <= 1e-13 and abs(p1 - F.plaquette(ref)) <= 1e-13
