"""The host regrid against the oracle's where neighbours wrap onto the leaf
itself or its siblings (one or two level-0 patches a side), over five levels
and tags that force long balance closures."""
import numpy as np
import pytest

import oracle
import paper_2205_07572_amd as af


@pytest.mark.parametrize("seed", [0, 1])
@pytest.mark.parametrize("n0x,n0y", [(1, 1), (1, 3), (2, 1), (2, 2), (5, 3)])
def test_regrid_matches_oracle(n0x, n0y, seed):
    lmax, m = 4, 8
    rng = np.random.default_rng(100 * n0x + 10 * n0y + seed)
    ctx = af.Context(af.Problem(eq=af.ADVECTION, prec=af.FP64, m=m, n0x=n0x, n0y=n0y, lmax=lmax, a=1.0, b=0.5))
    leaves = [(0, i, j) for j in range(n0y) for i in range(n0x)]
    h, o = af.Hierarchy(ctx, leaves), oracle.Hier(0, m, n0x, n0y, lmax)
    o.set_leaves(leaves)
    for it in range(12):
        n = len(h)
        tags = np.where(rng.random(n) < 0.7, -1, 0).astype(np.int8)
        if it % 3 != 2:  # few refinements, at the finest leaves
            tags[:] = 0
            tags[rng.integers(max(0, n - 8), n, 2)] = 1
        h = h.regrid(tags)
        o.regrid(tags)
        assert h.leaves() == [tuple(map(int, q)) for q in o.leaves()]
        np.testing.assert_array_equal(h.side_relations(), o.side_relations())
