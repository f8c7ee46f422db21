"""Workspace sizes of plans (host only): nothing is reserved that no kernel of
the plan reads or writes."""
import pytest

from paper_1510_03110_amd import rs


def _size(dims, **kw):
    plan = rs.rs_plan_create(dims, **kw)
    n = rs.rs_plan_workspace_size(plan)
    rs.rs_plan_destroy(plan)
    return n


@pytest.mark.parametrize("nx,nu", [(16, 8), (16, 1), (32, 5), (32, 15)])
def test_inputs_padded_in_the_kernels_have_no_copies(nx, nu):
    """A FP64 plan for the fused solve alone pads its inputs on load: it needs
    the workspace of 16 inputs, and a padding job's descriptor an instance."""
    count = 7
    full = _size([(nx, 16, 500)] * count, Ns=64, branch=4)
    assert full <= _size([(nx, nu, 500)] * count, Ns=64, branch=4) <= full + 256 * (count + 1)
    # plans that make the copies still have room for them
    copies = 8 * 500 * (2 * nx * 16 + 16 * 16 + 2 * 16) * count
    for kw in (dict(precision=rs.RS_MIXED_FP32), dict(flags=rs.RS_PLAN_FACTORED)):
        assert _size([(nx, nu, 500)] * count, Ns=64, branch=4, **kw) >= \
            _size([(nx, 16, 500)] * count, Ns=64, branch=4, **kw) + copies - 8 * 500 * 4 * 16 * count
