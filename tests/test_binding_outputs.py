"""The binding allocates only the outputs it is not given (no GPU: the allocator is replaced)."""

import pytest

import paper_2609_32197_amd as sp


def test_outputs_are_made_only_where_missing(monkeypatch):
    made = []
    monkeypatch.setattr(sp, "_empty", lambda shape, dtype, like: made.append((shape, dtype)) or "new")
    given = {"K_packed": "mine", "extra": 1}
    o = sp._outputs(given, None, demand=((2, 1), "i64"), K_packed=((8, 4, 4), "bf16"))
    assert o == {"K_packed": "mine", "extra": 1, "demand": "new"}
    assert made == [((2, 1), "i64")] and given == {"K_packed": "mine", "extra": 1}


def test_geometry_sizes_follow_the_fields():
    g = sp.Geometry(2, 1000, 64, 64, 3, 9, sp.BF16)
    assert (g.n, g.nq, g.W) == (16, 6, 1) and (g.n, g.nq, g.W) == (16, 6, 1)
    assert g == sp.Geometry(2, 1000, 64, 64, 3, 9, sp.BF16) and len({g, g}) == 1
    with pytest.raises(AttributeError):
        g.L = 5
