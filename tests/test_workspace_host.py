"""Workspace sizes (a host computation): beside the three state arrays a
handle holds tables of a few planes of the grid, reduction buffers and the
response samples' trace partials, of which large batches buffer fewer."""

import pytest

from paper_1706_09590_amd import inputs, qhfpe


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ns,np_,nq,depth,batch", [
    (2, 32, 128, 0, 64), (2, 32, 128, 0, 4096), (2, 128, 128, 6, 1024), (2, 64, 200, 1, 300), (3, 96, 96, 2, 100),
    (3, 256, 256, 8, 16), (2, 48, 48, 3, 1), (2, 192, 192, 8, 64), (2, 24, 24, 3, 500)])
def test_the_partials_stay_small(ns, np_, nq, depth, batch, precision):
    """The trace partials: at most 2 MiB, or 256 samples of one partial per 16
    columns (that is 128 bytes per column and member)."""
    d = inputs.model_dict(inputs.SMALL_ABSORPTION["model"], n_states=ns, nq=nq, np=np_, depth=depth)
    if ns == 3:
        d.update(poly=inputs.three_state_surfaces(0.3, 0.2), mu=[[0, 1, 0], [1, 0, 0], [0, 0, 0]])
    es = 8 if precision == "fp64" else 4
    states = 3 * batch * (depth + 1) * ns * ns * nq * np_ * es
    planes = (ns + ns * (ns - 1) // 2 + ns * (ns - 1) + (6 if ns == 3 else 5)) * nq * np_ * es
    blocks = ((depth + 1) * nq * np_ + 255) // 256
    reductions = 8 * batch * max(2 * blocks, 1024)
    members = batch * (64 + 4 * (depth + 2))
    if np_ == 24:  # one partial per 20 columns (tiles of ten groups, two columns each), always 256 samples
        partials = 256 * 8 * batch * -(-nq // 20)
    else:
        partials = max(2 * 2**20, 128 * nq * batch)
    fixed = 512 * 1024  # small tables and alignment
    assert qhfpe.workspace_bytes(d, batch, precision) <= states + planes + reductions + members + partials + fixed
