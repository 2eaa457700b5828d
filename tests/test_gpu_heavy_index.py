"""Rows at the edges of the heavy-row indexes: degrees one below a unit, exactly one unit, and the largest with two units, where
the lists of all rows together are as long as the build allows for.  Both orders of a layer against the oracle; the
fp32 tolerances of the parity tests."""
import numpy as np
import pytest

from paper_2201_02791_amd import synth

pytestmark = pytest.mark.gpu


def ring(n, R, k):
    """Every vertex has k edges out and k in: their heads, relations (in turn) and tails."""
    i, j = (x.ravel() for x in np.meshgrid(np.arange(n), np.arange(k), indexing="ij"))
    return i.astype(np.int32), (j % R).astype(np.int32), ((i + 1 + j % (n - 1)) % n).astype(np.int32)


# one relation: runs, destinations and sources of 255 .. 1022 edges; many: 63 .. 127 groups per source, 255 .. 511 runs per destination
@pytest.mark.parametrize("n,R,k", [(24, 1, 255), (24, 1, 256), (24, 1, 511), (9, 32, 32), (9, 63, 63), (9, 64, 63), (7, 128, 128), (7, 255, 255)])
@pytest.mark.parametrize("order", ["ORDER_PROJECT_FIRST", "ORDER_RELATION_WEIGHTS"])
def test_degrees_at_the_edges_of_units(orc, n, R, k, order):
    from paper_2201_02791_amd import binding
    from gpu_util import assert_partition_equal, assert_step_close, gpu_step, oracle_step
    print("[case] heavy", n, R, k, order, flush=True)
    head, rel, tail = ring(n, R, k)
    spec = synth.scaled(synth.WORKLOADS[0], name="ring", seed=6, n_entities=n, n_relations=R, n_triples=len(head), d=32, n_bases=4,
                        n_pos=64, n_neg=2, n_parts=1, part_id=0, acts=[0, 0])
    gp, ts, params, pos = gpu_step(spec, head, rel, tail, order=getattr(binding, order))
    op, res = oracle_step(orc, spec, head, rel, tail, params, pos)
    assert_partition_equal(gp, op)
    assert gp.max_in_degree == gp.max_out_degree == 2 * k
    assert_step_close(ts, res, 1e-5, 1e-4)
