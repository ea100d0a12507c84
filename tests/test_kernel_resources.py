"""LDS layout and scratch of kernels in the built library, as the compiler recorded them."""
import pytest

import _kernels
import paper_2604_24666_amd as P


@pytest.fixture(scope="module")
def kernels():
    return _kernels.kernels(P.LIB_PATH)


def _named(kernels, part):
    found = {n: k for n, k in kernels.items() if part in n}
    assert found, part
    return found


def test_pairs_in_dynamic_lds_are_aligned(kernels):
    """The table-gradient fill reads 8-byte pairs from its dynamic LDS, which starts where the static part
    ends."""
    for name, k in _named(kernels, "9k_tg_fill").items():
        assert k["lds"] % 8 == 0, (name, k)
