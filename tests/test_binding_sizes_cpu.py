"""The binding's sizes by the values of (params, shape) equal the library's own
queries, follow changes of a structure in place, and stay bounded."""

import pytest

from paper_2609_19702_amd import binding as B


def expect(p, s):
    L = B.state_layout(p, s)
    return (B.OK, B.window_logits_count(p, s) * 4, B.plan_bytes(p, s), L.bytes if L.cap else 0)


def test_sizes_follow_the_values():
    p, s = B.make_params(32, 16, 16, 64, 13), B.make_shape(1, 8, 8, 64)
    assert B._sizes(p, s) == expect(p, s) == B._sizes(p, s)
    p.n_att, s.batch = 20, 3  # the same objects, other values
    assert B._sizes(p, s) == expect(p, s)
    p.mode = B.MODE_DENSE
    assert B._sizes(p, s) == expect(p, s) and B._sizes(p, s)[3] == 0


def test_sizes_of_an_invalid_call_and_bound():
    bad = B.make_params(32, 16, 16, 64, 65)
    s = B.make_shape(1, 8, 8, 64)
    assert B._sizes(bad, s) == (B.ERR_INVALID_ARG, 0, 0, 0)
    with pytest.raises(B.DSAError):
        B._need_state(B._sizes(bad, s), None)
    for i in range(B._SIZES_MOST + 10):
        B._sizes(B.make_params(i, 16, 16, 64, 13), s)
    assert len(B._SIZES) <= B._SIZES_MOST
