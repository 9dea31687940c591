"""The F32C adjoint walks on FP32 particles, each of them: 8 targets a team
(n <= 7168), teams of 16, 8 and 4 wavefronts for 64 targets (up to 16384, 49152 and
1048576), one wavefront for 64 above.  (FP64 particles take the single-group walk in
F32C, whatever n is; it is checked here as well.)  The sets bring zero masses, cells
that several particles share, and wavefronts that straddle clumps far apart.
Bars: tests/bars.py."""
import numpy as np
import pytest

import oracle
import workloads
from bars import check_errors, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CENTRES = np.array([[x, y, z] for x in (0, 3) for y in (0, 5) for z in (0, 9)], float)


def _set(name, n, dtype):
    g = np.random.default_rng(n)
    if name == "plummer":  # a tenth without mass, and an corner of cells without any
        pos, m = workloads.plummer(n, 3, mass=workloads.lognormal_masses(n, 4))
        m[g.permutation(n)[:n // 10]] = 0.0
        m[(pos > 0.3).all(1)] = 0.0
    elif name == "clumps":
        pos, m = workloads.clumps(n // 8 + 1, CENTRES, 0.02, 5)
        k = g.permutation(len(pos))[:n]
        pos, m = pos[k], m[k]
        pos[::50] += g.normal(0, 4.0, pos[::50].shape)
    else:  # a twentieth of the particles at 400 places, 22 at one
        pos, m = g.random((n, 3)), np.full(n, 1.0 / n)
        k = g.permutation(n)[:n // 20]
        pos[k] = pos[:min(400, n // 2)][g.integers(0, min(400, n // 2), len(k))]
        pos[n // 3:n // 3 + 21] = pos[0]
    assert len(pos) == n
    return pos.astype(dtype), m.astype(dtype)


def _run(pos, m, seed):
    d = torch.device("cuda:0")
    g = np.random.default_rng(seed)
    ga, gp = (g.standard_normal(s).astype(np.float32) for s in ((len(pos), 3), len(pos)))
    return torch.from_numpy(pos).to(d), torch.from_numpy(m).to(d), torch.from_numpy(ga).to(d), torch.from_numpy(gp).to(d), ga, gp


@pytest.mark.parametrize("name", ["plummer", "clumps", "dups"])
@pytest.mark.parametrize("n,dtype", [(n, np.float32) for n in (65, 3001, 9001, 20001, 50001)] + [(9001, np.float64), (50001, np.float64)])
def test_gradients_match_oracle(name, n, dtype):
    import paper_2412_01733_amd as tc
    print("case", name, n, dtype.__name__, flush=True)
    pos, m = _set(name, n, dtype)
    p, mm, ga, gp, na, npot = _run(pos, m, n)
    theta, eps = 0.7, 0.01
    _, _, tree = tc.forces(p, mm, theta, eps)
    assert (name == "dups") == (tree.stats()["n_multi_leaves"] > 0)
    gx, gm = tree.backward(ga, gp)
    T = oracle.Tree(pos, m)
    ox, om = T.frozen_adjoint(T.lists(theta), eps, na, npot)
    for what, a, b in (("dL/dx", gx, ox), ("dL/dm", gm, om)):
        check_errors(rel_err(a.cpu().numpy(), b), "f32c", what=what, per_target=False)


@pytest.mark.parametrize("name", ["plummer", "clumps", "dups"])
@pytest.mark.parametrize("n", [7168, 7169, 16384, 16385, 49152, 49153, 1048576, 1048577])
def test_walks_match_the_replay_of_lists(name, n):
    """Both sides of the lines, against the replay of stored lists on the same tree
    (walk.hip; here, with FP32 particles, another kernel): the same terms, so the sums
    differ by rounding only."""
    import paper_2412_01733_amd as tc
    print("case", name, n, flush=True)
    pos, m = _set(name, n, np.float32)
    p, mm, ga, gp, _, _ = _run(pos, m, n)
    _, _, tree = tc.forces(p, mm, 0.7, 0.01, store_lists=True)
    assert tree.stats()["lists_stored"]
    rx, rm = tree.backward(ga, gp)
    tree.forces(0.7, 0.01)
    gx, gm = tree.backward(ga, gp)
    for what, a, b in (("dL/dx", gx, rx), ("dL/dm", gm, rm)):
        check_errors(rel_err(a.cpu().numpy(), b.cpu().numpy()), "f32c", what=what, per_target=False)
