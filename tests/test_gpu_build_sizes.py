"""The build at the sizes where its kernels change hands: one tile of the small
sort (2048) and its merges (8, 64 tiles; odd tails), one block of the tree
kernels (1024), and the radix sort above 2^19; every table against the oracle,
bit for bit.  Duplicated keys check the stability of the merges and leaves of
several particles on both sides of a block's edge."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dups(n, seed):
    """A third of the particles share 7 positions (shuffled, so that their runs
    meet in the merges and their leaves span blocks)."""
    g = np.random.default_rng(seed)
    pos = g.random((n, 3))
    k = g.permutation(n)[:n // 3]
    pos[k] = pos[:7][g.integers(0, 7, len(k))]
    return pos.astype(np.float32), np.full(n, 1.0 / n, np.float32)


CASES = [(n, "plummer") for n in (1023, 1024, 1025, 2047, 2048, 2049, 4097, 16384, 16385, 131073, 524288, 524289)]
CASES += [(n, "dups") for n in (2050, 20000, 140001, 600001)]
# the radix sort's tiles change from 2048 to 3072 keys at 5 * 2^18 (whole tiles, a tail of one key, eighths of unequal length)
CASES += [(1310719, "plummer"), (1310720, "plummer"), (1310721, "dups"), (3072 * 431, "plummer")]

# the upward pass: the whole tree in one workgroup up to 4096 particles, parts of 1024 up to 2^18, of 2048 up to
# 5 * 2^17, level by level above (leaves and nodes that cross parts, a lone particle in the last part)
CASES += [(n, k) for n in (4096, 262144, 262145, 655360, 655361) for k in ("plummer", "dups")]
CASES += [(2, "plummer"), (1025, "dups"), (3073, "dups"), (260097, "plummer"), (264193, "dups")]


@pytest.mark.parametrize("n,kind", CASES)
def test_tables_match_oracle(n, kind):
    import paper_2412_01733_amd as tc
    print("case", n, kind, flush=True)
    pos, m = workloads.plummer(n, 40 + n % 97, dtype=np.float32) if kind == "plummer" else _dups(n, n)
    d = torch.device("cuda:0")
    t = tc.Tree()
    t.build(torch.from_numpy(pos).to(d), torch.from_numpy(m).to(d)).moments()
    ex = {k: v.cpu().numpy() for k, v in t.export().items()}
    T = oracle.Tree(pos, m)
    ok, op = T.sorted()
    nd = T.nodes()
    assert (ex["keys"].view(np.uint64) == ok).all() and (ex["perm"].astype(np.int64) == op).all()
    assert len(ex["level"]) == len(nd["level"])
    for k in ("level", "first", "count"):
        assert (ex[k].astype(np.int64) == nd[k]).all(), k
    assert (ex["mass"] == nd["mass"]).all() and (ex["com"] == nd["com"]).all()
    st = t.stats()
    assert st["n_leaves"] == int((nd["nchild"] == 0).sum())
    assert st["n_multi_leaves"] == int(((nd["nchild"] == 0) & (nd["count"] > 1)).sum())
    order = t.target_order().cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(n))
