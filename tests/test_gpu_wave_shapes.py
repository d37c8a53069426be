"""The wave variant's launch shapes (columns per wave, components in flight,
workgroup size, non-temporal stores), which are chosen by the launch's size:
a member's states and traces are the same bits in a batch of every size, and
the smallest batch agrees with the oracle.  Bars as in test_gpu_parity.py
(FP64 1e-12 per operator application)."""

import numpy as np
import pytest

from helpers import oracle_model
from oracle import qhfpe_oracle as O
from paper_1706_09590_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1706_09590_amd import qhfpe  # noqa: E402

NPS = [32, 48, 64, 96, 128, 192, 256]
GROUPS = {32: 4, 48: 4, 64: 1, 96: 2, 128: 1, 192: 1, 256: 1}


def model(ns, np_, nq=10, depth=1, **kw):
    kw.update(n_states=ns, nq=nq, np=np_, depth=depth, dt=0.001)
    if ns == 3:
        kw.update(poly=inputs.three_state_surfaces(0.3, 0.2), mu=[[0, 1, 0], [1, 0, 0], [0, 0, 0]])
    return inputs.model_dict(inputs.SMALL_ABSORPTION["model"], **kw)


def run(d, batch, precision, q_dependent):
    P = qhfpe.Propagator(d, batch=batch, precision=precision)
    try:
        if q_dependent:
            P.set_potential(lambda j, l, x: 0.5 * x * x + 3.0 * j if j == l else 0.3 * np.exp(-0.2 * x * x))
        P.init_thermal(1.0)
        P.apply_dipole()
        tr = P.step(2, 1).cpu().numpy()
        return [(tr[m], P.get_state(member=m).cpu().numpy()) for m in (0, batch - 1)]
    finally:
        P.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ns,q_dependent", [(2, False), (2, True), (3, False)])
@pytest.mark.parametrize("np_", NPS)
def test_results_do_not_depend_on_the_launch_shape(np_, ns, q_dependent, precision):
    d = model(ns, np_)
    per_member = 2 * -(-d["nq"] // GROUPS[np_])  # waves with one column per lane group
    reals = 2 * ns * ns * d["nq"] * np_
    nt = int(256 * 2**20 / (3 * reals * (8 if precision == "fp64" else 4))) + 1  # non-temporal stores
    ref = run(d, 1, precision, q_dependent)[0]
    for batch in sorted({-(-w // per_member) for w in (900, 1700, 3500, 7400, 13500)} | {nt}):
        for tr, st in run(d, batch, precision, q_dependent):
            np.testing.assert_array_equal(tr, ref[0], err_msg=str(batch))
            np.testing.assert_array_equal(st, ref[1], err_msg=str(batch))


@pytest.mark.parametrize("ns", [2, 3])
@pytest.mark.parametrize("np_", NPS)
def test_rhs_parity_with_a_sign_change_inside_a_lane(np_, ns):
    """One column past the lane groups' last, unsmoothed data, and a p grid
    whose sign change falls between the nodes of one lane."""
    d = model(ns, np_, nq=GROUPS[np_] + 5, depth=2, p_min=-7.9, p_max=8.1)
    W = inputs.random_hierarchy(2, ns, d["nq"], np_, seed=60 + np_ + ns, smooth=False)
    P = qhfpe.Propagator(d, batch=1, precision="fp64")
    try:
        P.set_state(torch.from_numpy(W[None]))
        P.apply_rhs()
        got = P.get_state().cpu().numpy()[0]
    finally:
        P.close()
    ref = O.rhs(oracle_model(d), W)
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)
