"""The walks with 8 or 16 targets a wavefront or a team of wavefronts for 64
targets (no counting, no stored lists) against the FP64 oracle, at sizes around one wavefront's targets,
with multi-particle leaves, the direct sum, and on both sides of the sizes at
which the library changes the number of targets (there against the 64-target
walk, which the counting walk always uses: the decisions are the same, so the
outputs may differ by rounding only).  Bars: tests/bars.py."""
import numpy as np
import pytest

import oracle
import workloads
from bars import check_errors, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dups(n, seed):
    g = np.random.default_rng(seed)
    pos = g.random((n, 3))
    pos[n // 3:n // 3 + 21] = pos[0]  # a leaf of 22 particles
    pos[n // 2:n // 2 + 3] = pos[5] + 1e-9
    return pos, np.full(n, 1.0 / n)


CASES = [("n%d" % n, lambda n=n: workloads.plummer(n, 500 + n), 0.6, 0.05) for n in (2, 7, 8, 9, 17, 63, 65, 1001, 12301)]
CASES += [
    ("dups4097", lambda: _dups(4097, 4), 0.6, 0.001),
    ("direct3001", lambda: workloads.plummer(3001, 77), 0.0, 0.01),
    ("disc", lambda: workloads.disc_galaxy(5000, 1003, 5, dtype=np.float32)[0::2], 1.2, 0.02),
]


def _gpu(pos, m):
    d = torch.device("cuda:0")
    return torch.from_numpy(np.ascontiguousarray(pos)).to(d), torch.from_numpy(np.ascontiguousarray(m)).to(d)


@pytest.mark.parametrize("walk", ["f32c", "f64"])
@pytest.mark.parametrize("name,make,theta,eps", CASES, ids=[c[0] for c in CASES])
def test_split_walks_match_oracle(name, make, theta, eps, walk):
    import paper_2412_01733_amd as tc
    print("case", name, walk, flush=True)
    pos, m = make()
    p, mm = _gpu(pos, m)
    _, _, tree = tc.forces(p, mm, theta, eps, walk=walk, count=True)
    counts = tree.interaction_counts().cpu().numpy().astype(np.int64)
    acc, pot = tree.forces(theta, eps, walk=walk)
    T = oracle.Tree(pos, m)
    ra, rp, nint = T.forces(theta, eps)
    same = counts == nint
    check_errors(rel_err(acc.cpu().numpy(), ra), walk, same, "acc")
    check_errors(rel_err(pot.cpu().numpy(), rp), walk, same, "pot")
    again, _ = tree.forces(theta, eps, walk=walk)
    assert torch.equal(acc, again)
    g = np.random.default_rng(11)
    ga, gp = g.standard_normal(pos.shape), g.standard_normal(len(pos))
    gx, gm = tree.backward(torch.from_numpy(ga).to(p.device), torch.from_numpy(gp).to(p.device))
    ox, om = T.frozen_adjoint(T.lists(theta), eps, ga, gp)
    check_errors(rel_err(gx.cpu().numpy(), ox), walk, what="dL/dx", per_target=False)
    check_errors(rel_err(gm.cpu().numpy(), om), walk, what="dL/dm", per_target=False)
    st = tree.stats()
    md = np.asarray(m, np.float64)
    assert abs(st["sum_m_abs_a"] / (md * np.linalg.norm(ra, axis=1)).sum() - 1) < 1e-6


@pytest.mark.parametrize("walk,n", [(w, n) for w in ("f32c", "f64") for n in (12288, 12289, 24576, 24577, 81920, 81921)] + [
                                    ("f32c", 40960), ("f32c", 40961), ("f32c", 98304), ("f32c", 98305), ("f32c", 524288),
                                    ("f32c", 524289), ("f64", 40961), ("f64", 131072), ("f64", 131073), ("f64", 786432),
                                    ("f64", 786433)])
def test_both_sides_of_the_lines(walk, n):
    import paper_2412_01733_amd as tc
    print("case", walk, n, flush=True)
    p, mm = _gpu(*workloads.plummer(n, 9, dtype=np.float32))
    tree = tc.Tree()
    tree.build(p, mm).moments()
    a64, p64 = tree.forces(0.7, 0.01, walk=walk, count=True)
    acc, pot = tree.forces(0.7, 0.01, walk=walk)
    check_errors(rel_err(acc.cpu().numpy(), a64.cpu().numpy()), walk, what="acc")
    check_errors(rel_err(pot.cpu().numpy(), p64.cpu().numpy()), walk, what="pot")


@pytest.mark.parametrize("walk", ["f32c", "f64"])
@pytest.mark.parametrize("name", ["plummer", "clumps", "dups", "wide_theta"])
def test_wide_walk_matches_oracle(name, walk):
    """The 64-target walk as large inputs take it (above the lines it is the same
    kernel that counts, so a counting call stands for it here), with masks of
    every density: compact clumps seen from afar, outliers whose wavefronts are
    spread out, leaves of several particles, theta > 1/sqrt(3)."""
    import paper_2412_01733_amd as tc
    print("case", name, walk, flush=True)
    theta, eps = 0.5, 0.005
    if name == "plummer":
        pos, m = workloads.plummer(30011, 3)
    elif name == "clumps":
        ctr = np.array([[x, y, z] for x in (0, 3) for y in (0, 5) for z in (0, 9)], float)
        pos, m = workloads.clumps(1501, ctr, 0.02, 5)
        pos[::50] += np.random.default_rng(1).normal(0, 4.0, pos[::50].shape)
    elif name == "dups":
        pos, m = _dups(9001, 8)
        eps = 0.001
    else:
        pos, m = workloads.plummer(12001, 4)
        theta = 1.3
    p, mm = _gpu(pos, m)
    acc, pot, tree = tc.forces(p, mm, theta, eps, walk=walk, count=True)
    T = oracle.Tree(pos, m)
    ra, rp, nint = T.forces(theta, eps)
    counts = tree.interaction_counts().cpu().numpy().astype(np.int64)
    assert np.mean(counts != nint) < (0.01 if walk == "f32c" else 1e-3)
    check_errors(rel_err(acc.cpu().numpy(), ra), walk, counts == nint, "acc")
    check_errors(rel_err(pot.cpu().numpy(), rp), walk, counts == nint, "pot")
    again, _, _ = tc.forces(p, mm, theta, eps, walk=walk, count=True)
    assert torch.equal(acc, again)


@pytest.mark.parametrize("walk,n", [("f32c", 12288), ("f32c", 12289), ("f32c", 300007), ("f32c", 1048576), ("f32c", 1048577),
                                    ("f64", 16384), ("f64", 16385), ("f64", 393216), ("f64", 393217)]
                         + [(w, n) for w in ("f32c", "f64") for n in (6144, 6145, 7168, 7169, 49152, 49153)] + [("f32c", 16385), ("f64", 6151)])
@pytest.mark.parametrize("name", ["plummer", "clumps", "dups"])
def test_wide_adjoint_matches_replay(name, walk, n):
    """The adjoint walks against the replay of stored lists on the same
    tree (another kernel, the same terms): they may differ by rounding and, in
    F32C, by nothing else, since the decisions are the same."""
    import paper_2412_01733_amd as tc
    print("case", name, walk, n, flush=True)
    g = np.random.default_rng(n)
    eps = 0.01
    if name == "plummer":
        pos, m = workloads.plummer(n, 3, mass=workloads.lognormal_masses(n, 4))
    elif name == "clumps":
        pos, m = workloads.clumps(n // 8 + 1, np.array([[x, y, z] for x in (0, 3) for y in (0, 5) for z in (0, 9)], float), 0.02, 5)
        pos[::50] += g.normal(0, 4.0, pos[::50].shape)
    else:
        pos, m = _dups(n, 8)
        k = g.permutation(n)[:n // 20]
        pos[k] = pos[:400][g.integers(0, 400, len(k))]
    p, mm = _gpu(pos, m)
    n = len(pos)
    dt = torch.float32 if walk == "f32c" else torch.float64
    ga, gp = (torch.from_numpy(g.standard_normal(s)).to(p.device, dt) for s in ((n, 3), n))
    acc, pot, tree = tc.forces(p, mm, 0.7, eps, walk=walk, store_lists=True)
    assert tree.stats()["lists_stored"]
    rx, rm = tree.backward(ga, gp)
    a2, p2 = tree.forces(0.7, eps, walk=walk)
    gx, gm = tree.backward(ga, gp)
    for what, a, b in (("acc", a2, acc), ("pot", p2, pot), ("dL/dx", gx, rx), ("dL/dm", gm, rm)):
        check_errors(rel_err(a.cpu().numpy(), b.cpu().numpy()), walk, what=what, per_target=False)


@pytest.mark.parametrize("walk", ["f32c", "f64"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 4099])
def test_direct_kernel_matches_oracle(n, walk):
    """theta = 0 around a block's targets, a run of sources and the 16 runs of a block."""
    import paper_2412_01733_amd as tc
    pos, m = workloads.plummer(n, 70 + n)
    p, mm = _gpu(pos, m)
    acc, pot, _ = tc.forces(p, mm, 0.0, 0.01, walk=walk)
    if n == 1:
        assert (acc == 0).all() and (pot == 0).all()
        return
    ra, rp = oracle.direct(pos, m, 0.01)
    check_errors(rel_err(acc.cpu().numpy(), ra), walk, what="acc")
    check_errors(rel_err(pot.cpu().numpy(), rp), walk, what="pot")


@pytest.mark.parametrize("walk", ["f32c", "f64"])
def test_direct_sum_with_shared_cells_takes_the_walk(walk):
    """Leaves of several particles need FP64 separations: theta = 0 then walks."""
    import paper_2412_01733_amd as tc
    pos, m = _dups(1500, 6)
    p, mm = _gpu(pos, m)
    acc, pot, tree = tc.forces(p, mm, 0.0, 0.001, walk=walk)
    assert tree.stats()["n_multi_leaves"] > 0
    ra, rp = oracle.direct(pos, m, 0.001)
    check_errors(rel_err(acc.cpu().numpy(), ra), walk, what="acc")
    check_errors(rel_err(pot.cpu().numpy(), rp), walk, what="pot")


@pytest.mark.parametrize("walk", ["f32c", "f64"])
@pytest.mark.parametrize("name", ["one", "coincident", "pair", "chain"])
def test_climb_to_the_root(name, walk):
    """Gradients where the way from a particle's leaf to the root has no step (the
    root is the leaf), one, or all 21 (particles 2^-20 of the cube apart)."""
    import paper_2412_01733_amd as tc
    pos = {"one": [[0.5, 0.25, 0.125]], "coincident": [[0.5, 0.25, 0.125]] * 5, "pair": [[0.0, 0.0, 0.0], [1.0, 0.5, 0.25]],
           "chain": [[0.0, 0.0, 0.0], [2.0 ** -20, 0.0, 0.0], [0.0, 2.0 ** -21, 0.0], [1.0, 1.0, 1.0]]}[name]
    pos = np.array(pos)
    n = len(pos)
    m = np.arange(1.0, n + 1) / n
    p, mm = _gpu(pos, m)
    _, _, tree = tc.forces(p, mm, 0.7, 0.5, walk=walk)
    g = np.random.default_rng(3)
    ga, gp = g.standard_normal((n, 3)), g.standard_normal(n)
    gx, gm = tree.backward(torch.from_numpy(ga).to(p.device), torch.from_numpy(gp).to(p.device))
    T = oracle.Tree(pos, m)
    ox, om = T.frozen_adjoint(T.lists(0.7), 0.5, ga, gp)
    # a few terms of order |g| m / eps^3 = O(10), each within a few roundings
    tol = 1e-5 if walk == "f32c" else 1e-13
    assert np.abs(gx.cpu().numpy() - ox).max() <= 10 * tol and np.abs(gm.cpu().numpy() - om).max() <= 10 * tol


@pytest.mark.parametrize("n", [9001, 16385])
def test_gradients_of_fp64_particles_are_those_of_the_single_group_walk(n):
    """FP32 terms, FP64 particles: the walk that lists of more than 8192 records a
    wavefront (theta = 0) fall back to, so the same sums with that flag as without
    (only the order of the FP64 atomics differs, which flips few FP32 roundings)."""
    import paper_2412_01733_amd as tc
    pos, m = workloads.plummer(n, 5, mass=workloads.lognormal_masses(n, 6))
    p, mm = _gpu(pos, m)
    assert p.dtype == torch.float64
    g = np.random.default_rng(n)
    ga, gp = (torch.from_numpy(g.standard_normal(s)).to(p.device) for s in ((n, 3), n))
    _, _, tree = tc.forces(p, mm, 0.0, 0.01, store_lists=True)
    assert tree.stats()["lists_stored"]
    rx, rm = tree.backward(ga, gp)
    tree.forces(0.0, 0.01)
    gx, gm = tree.backward(ga, gp)
    for a, b in ((gx, rx), (gm, rm)):
        assert (a.double() - b.double()).norm() <= 1e-8 * b.double().norm()
