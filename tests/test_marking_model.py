"""Host model of how a wave marks the first r distinct values of a word stream
(CPU): the removed hits of a dense leaf (Algorithm B, Sec. 2) and the values of
a small leaf that expects repeats.

While h values are marked, the next r - h words are taken, no further than the
256 words in registers, and the value of every one that is not void is marked
by an atomic OR.  So many words hold no more new values than are missing:
nothing is marked that the first r distinct values in stream order (the
definition, which the oracle implements) do not hold, whatever order the atomics
are served in.  The model plays each step in random orders and counts as the
kernels do, a lane whose bit was clear before its own OR.
"""
import random

import pytest


def first_distinct(values, r):
    out = []
    for v in values:
        if v is not None and v not in out:
            out.append(v)
            if len(out) == r:
                break
    return set(out)


def marked(values, r, rng):
    """The kernels' selection and the words they read."""
    marks, have, t = set(), 0, 0
    while have < r:
        t0 = t & ~255
        end = min(t + (r - have), t0 + 256)
        for j in range(4):  # lane l holds words t0 + 4 l + j
            lanes = [t0 + 4 * lane + j for lane in range(64)]
            for i in rng.sample(lanes, 64):
                v = values[i] if t <= i < end else None
                if v is not None:
                    have += v not in marks
                    marks.add(v)
        t = end
    return marks, t


@pytest.mark.parametrize("size,r,void_rate", [
    (100, 30, 0.0), (4000, 200, 0.0), (64, 63, 0.0), (64, 64, 0.0), (5, 5, 0.3), (1, 1, 0.0),
    (3000, 150, 0.45), (16000, 1000, 0.0), (2003, 1000, 0.4), (600, 257, 0.0), (600, 256, 0.2),
])
def test_marks_are_the_first_distinct_values(size, r, void_rate):
    rng = random.Random(1000 * size + r)
    for _trial in range(20):
        values = [None if rng.random() < void_rate else rng.randrange(size)
                  for _ in range(256 * (8 + 12 * r // 64))]
        want = first_distinct(values, r)
        assert len(want) == r
        for _order in range(2):
            got, read = marked(values, r, rng)
            assert got == want
            assert read <= len(values)


def test_words_read_end_where_the_last_value_is_found():
    # no word past the one that completes the set is ever marked
    values = [3, 3, 3, 7] + [9] * 508
    got, read = marked(values, 2, random.Random(1))
    assert got == {3, 7} and read <= 5
