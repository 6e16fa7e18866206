"""Host rules that choose between two ways of doing the same call."""
import itertools

from . import routes


def test_ranges_overlap_as_sets_of_bytes():
    r = routes.load()
    for p, q in itertools.product(range(8), repeat=2):
        for pn, qn in itertools.product(range(5), repeat=2):
            want = bool(set(range(p, p + pn)) & set(range(q, q + qn)))
            assert bool(r.ranges_overlap(16 + p, pn, 16 + q, qn)) == want, (p, pn, q, qn)
    top = 2 ** 64 - 16
    assert r.ranges_overlap(top, 16, top + 15, 1) and not r.ranges_overlap(top, 15, top + 15, 1)


def test_a_kernel_writes_only_memory_of_the_one_device():
    """Memory, handle and current device: a handle of one device may not write a peer's memory by a kernel, whichever
    of the two is current, nor may a handle whose stream is another device's (-1)."""
    r = routes.load()
    for memory, handle, current in itertools.product((0, 1), (-1, 0, 1), (0, 1)):
        assert bool(r.one_device(memory, handle, current)) == (memory == handle == current)
