"""Infinite upstream gradients (an overflowed loss scale): what the plain sums of
the oracle make infinite stays infinite with the same sign, what they make
undefined stays undefined, in both walks and through every adjoint walk."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("walk,dtype,n", [("f32c", np.float32, 3000), ("f32c", np.float32, 9001), ("f32c", np.float32, 60001),
                                          ("f32c", np.float64, 3000), ("f64", np.float64, 3000), ("f64", np.float64, 9001),
                                          ("f64", np.float32, 60001)])
def test_infinite_potential_gradient(walk, dtype, n):
    """dL/dphi of one target is infinite: every other particle is in one of its
    terms, so dL/dx is infinite for all of them, away from or towards the target;
    the target's own sum holds both signs."""
    import paper_2412_01733_amd as tc
    print("case", walk, dtype.__name__, n, flush=True)
    pos, m = workloads.plummer(n, 7, dtype=dtype)
    g = np.random.default_rng(n)
    ga, gp = g.standard_normal((n, 3)), np.zeros(n)
    gp[5] = np.inf
    T = oracle.Tree(pos, m)
    ox, om = T.frozen_adjoint(T.lists(0.6), 0.01, ga, gp)
    assert np.isinf(np.delete(ox, 5, 0)).all() and np.isnan(ox[5]).all()
    d = torch.device("cuda:0")
    _, _, tree = tc.forces(torch.from_numpy(pos).to(d), torch.from_numpy(m).to(d), 0.6, 0.01, walk=walk)
    dt = torch.float32 if walk == "f32c" else torch.float64
    gx, gm = (v.double().cpu().numpy() for v in tree.backward(torch.from_numpy(ga).to(d, dt), torch.from_numpy(gp).to(d, dt)))
    # its mass is in none of its own terms
    assert np.isnan(gx[5]).all() and np.array_equal(np.isfinite(gm), np.isfinite(om))
    rest = np.delete(gx, 5, 0)
    assert np.isinf(rest).all(), np.isnan(rest).mean()
    # the sign is the oracle's wherever both take the particle in the same term (a target whose
    # opening test sits within rounding of its threshold may use another node)
    assert (rest == np.delete(ox, 5, 0)).mean() > 0.99
