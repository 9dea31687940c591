"""Handles used from several streams."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("others", [1, 3, 4, 6])
def test_free_waits_for_every_stream_the_handle_was_used_on(others):
    """A force evaluation is held up on one stream by work of the caller's; the tree is
    read on `others` more streams, which finish at once; freeing the handle waits for
    the first all the same (its buffers and its host mirror go to the next handle),
    and the next handle's diagnostics are its own."""
    import paper_2412_01733_amd as tc
    d = torch.device("cuda:0")
    pos, m = (torch.from_numpy(a).to(d) for a in workloads.plummer(3000, 5, dtype=np.float32))
    _, _, ref = tc.forces(pos, m, 0.5, 0.05)
    want = ref.stats()["momentum"]
    ref.free()
    slow, streams = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(others)]
    # everything once beforehand, so that first calls do not take the time of the wait below
    for s in [slow] + streams:
        with torch.cuda.stream(s):
            t = tc.Tree().build(pos, m).moments()
            t.forces(0.5, 0.05)
            t.target_order()
            t.free()
    begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    torch.cuda._sleep(1000)
    begin.record()
    torch.cuda._sleep(10_000_000)
    end.record()
    torch.cuda.synchronize()
    half_a_second = int(10_000_000 * 500.0 / begin.elapsed_time(end))
    tree = tc.Tree()
    with torch.cuda.stream(slow):
        tree.build(pos, m).moments()
        acc = torch.empty((3000, 3), device=d)
        slow.synchronize()
        torch.cuda._sleep(half_a_second)
        tree.forces(0.5, 0.05, potential=False, out=(acc, None))
        done = slow.record_event()
    for s in streams:
        with torch.cuda.stream(s):
            tree.target_order()
    assert not done.query()  # the case is what it says
    tree.free()
    assert done.query()
    nxt = tc.forces(pos, 2 * m, 0.5, 0.05)[2]
    got = nxt.stats()["momentum"]
    torch.cuda.synchronize()
    assert got == nxt.stats()["momentum"] and got == [4 * v for v in want]


@pytest.mark.parametrize("n", [700, 20000, 600001])
def test_export_only_reads_the_handle(n):
    """tc_tree_export takes a const handle: not a byte of the buffers it owns changes
    (so exports on several streams do not meet), and exports that run at once agree."""
    import paper_2412_01733_amd as tc
    from paper_2412_01733_amd import _lib
    d = torch.device("cuda:0")
    pos, m = (torch.from_numpy(a).to(d) for a in workloads.plummer(n, 6, dtype=np.float32))
    held = {}

    def alloc(nbytes, stream, ctx):
        t = torch.zeros(int(nbytes), dtype=torch.uint8, device=d)
        held[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, stream, ctx):
        held.pop(int(ptr), None)

    fa, ff = _lib.ALLOC_FN(alloc), _lib.FREE_FN(free)
    tc.Tree()  # installs torch's allocator, if it is the first
    lib = _lib.load()
    try:
        assert lib.tc_set_allocator(fa, ff, None) == _lib.TC_OK
        tree = tc.Tree()
        tree.build(pos, m).moments()
        tree.forces(0.5, 0.05)
        torch.cuda.synchronize()
        before = {p: t.clone() for p, t in held.items()}
        one = tree.export()
        torch.cuda.synchronize()
        assert before.keys() == held.keys()
        for p, t in held.items():
            assert torch.equal(before[p], t), int((before[p] != t).sum())
        out = []
        for s in (torch.cuda.Stream(), torch.cuda.Stream()):
            with torch.cuda.stream(s):
                out.append(tree.export())
        torch.cuda.synchronize()
        for e in out:
            assert all(torch.equal(e[k], one[k]) for k in one)
        tree.free()
    finally:
        assert lib.tc_set_allocator(_lib.ALLOC_FN(), _lib.FREE_FN(), None) == _lib.TC_OK
        tc.treecode.bind_torch_allocator()


def test_more_handles_than_the_pool_keeps():
    """Twelve handles at once (the pool of host mirrors keeps eight), freed out of
    order and made anew, each with its own diagnostics."""
    import paper_2412_01733_amd as tc
    d = torch.device("cuda:0")
    sets = [[torch.from_numpy(a).to(d) for a in workloads.plummer(500 + 7 * i, i, dtype=np.float32)] for i in range(12)]
    want = None
    for _ in range(3):
        trees = [tc.forces(p, m, 0.5, 0.05)[2] for p, m in sets]
        got = [t.stats()["momentum"] for t in trees]
        assert want is None or got == want
        want = got
        for i in (3, 0, 11, 5, 1, 2, 4, 10, 9, 8, 7, 6):
            trees[i].free()
