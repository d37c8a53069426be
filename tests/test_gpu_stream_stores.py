"""Stages that write non-temporally (state arrays past the library's limit)
give every member the bits it has in a batch of its own, which writes
through the caches; members of their own depths among them."""

import os
import re

import numpy as np
import pytest

from paper_1706_09590_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1706_09590_amd import qhfpe  # noqa: E402

NQ, DEPTH = 61, 7
BATHS = {0: (0.5, 1.0, 1.0), -1: (0.8, 0.7, 0.9)}


def limit_bytes():
    """The library's limit (qhfpe_handle::stream_out)."""
    src = os.path.join(os.path.dirname(qhfpe.__file__), "csrc", "qhfpe_api.cpp")
    m = re.search(r"kStreamBytes = ([0-9.]+) \* 1024 \* 1024;", open(src).read())
    return float(m.group(1)) * 2**20


def run(d, batch, precision, q_dependent, depths, members):
    P = qhfpe.Propagator(d, batch=batch, precision=precision)
    try:
        for m, bath in members.items():
            P.set_member_bath(m, *bath)
        for m, n in depths.items():
            P.set_member_depth(m, n)
        if q_dependent:
            P.set_potential(lambda j, l, x: 0.5 * x * x + 3.0 * j if j == l else 0.3 * np.exp(-0.2 * x * x))
        P.init_thermal(1.0)
        P.apply_dipole()
        tr = P.step(2, 1).cpu().numpy()
        return {m: (tr[m], P.get_state(member=m).cpu().numpy()) for m in members}
    finally:
        P.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ns,q_dependent", [(2, False), (2, True), (3, False)])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("np_", [32, 48, 64, 96, 128, 192, 256])
def test_streamed_members_equal_a_batch_of_one(np_, mixed, ns, q_dependent, precision):
    d = inputs.model_dict(inputs.SMALL_ABSORPTION["model"], n_states=ns, nq=NQ, np=np_, depth=DEPTH, dt=0.001)
    if ns == 3:
        d.update(poly=inputs.three_state_surfaces(0.3, 0.2), mu=[[0, 1, 0], [1, 0, 0], [0, 0, 0]])
    level = 3 * ns * ns * NQ * np_ * (8 if precision == "fp64" else 4)  # of the three state arrays
    # the last member has three levels of its own in a mixed batch
    batch = int(limit_bytes() / (level * (DEPTH + 1))) + 2
    last = batch - 1
    depths = {last: 2} if mixed else {}
    levels = batch * (DEPTH + 1) - (DEPTH - 2 if mixed else 0)
    assert levels * level > limit_bytes()
    got = run(d, batch, precision, q_dependent, depths, {0: BATHS[0], last: BATHS[-1]})
    for m, bath in ((0, BATHS[0]), (last, BATHS[-1])):
        own = {0: depths[m]} if m in depths else {}
        want = run(d, 1, precision, q_dependent, own, {0: bath})[0]
        np.testing.assert_array_equal(got[m][0], want[0])
        np.testing.assert_array_equal(got[m][1], want[1])
