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


def test_traversal_state_stays_in_registers(kernels):
    """Bin steps that update the walk in place through a selected address put it into scratch (16 bytes a
    lane in every kernel below).  The 64-ray waves at width 64 and the tracing with 16 lanes a ray use all
    the registers they are given and may spill 12 bytes, none of them the walk's."""
    for part, limit in (("7k_traceILi8E", 0), ("7k_traceILi16E", 12), ("7k_first", 0), ("7k_proxy", 0), ("13k_query_block", 0)):
        for name, k in _named(kernels, part).items():
            assert k["scratch"] <= limit, (name, k)
    for width, limit in ((16, 0), (32, 0), (64, 12)):
        for rays in (16, 64):
            for name, k in _named(kernels, f"7k_queryILi{width}ELi0ELi{rays}ELb0ELi2E").items():
                assert k["scratch"] <= limit, (name, k)
