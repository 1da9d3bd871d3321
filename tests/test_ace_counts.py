"""Descriptor counts and the rank-4 set from counting rules, at every size that
the grid ACE entry points take, against the oracle's explicit enumeration (its
rank-4 set from the rank of the symmetrised coupling coefficients)."""
import pytest

import oracle
import paper_2411_19617_amd as mala


@pytest.mark.parametrize("nmax4", [1, 2, 3])
@pytest.mark.parametrize("lmax4", [0, 1, 2, 3])
def test_rank4_set(nmax4, lmax4):
    want = [tuple(int(x) for x in d) for d in oracle.ace4_set(nmax4, lmax4)]
    assert [tuple(int(x) for x in d) for d in mala.ace4_list(nmax4, lmax4)] == want
    assert mala.ace4_count(nmax4, lmax4) == len(want)


@pytest.mark.parametrize("nmax", [1, 2, 3, 4])
def test_rank123_count(nmax):
    for lmax in range(5):
        assert mala.ace_count(nmax, lmax) == oracle.ace_count(nmax, lmax)
