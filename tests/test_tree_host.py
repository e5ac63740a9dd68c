"""Host-only test of the row that a tree draw belongs to (simgraph_tree.hip's own
division by the draws per row), up to the largest draw index."""
import ctypes as C
import random

import pytest

from tests.test_lsh_host import build


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    lib = C.CDLL(build(tmp_path_factory.mktemp("treemock"), "tree_host.cpp"))
    lib.tree_row_of_draw.restype = C.c_uint32
    lib.tree_row_of_draw.argtypes = [C.c_uint32, C.c_uint32]
    return lib


def test_row_of_a_draw(lib):
    top = (1 << 31) - 1
    rng = random.Random(1)
    sizes = {1, 2, 3, 5, 7, 10, 17, 641, 6700417, top} | {(1 << k) + o for k in range(1, 31) for o in (-1, 0, 1)}
    sizes |= {rng.randint(1, top) for _ in range(300)}
    for s in sizes:
        es = {0, 1, top, top - 1} | {rng.randint(0, top) for _ in range(30)}
        for q in (1, 2, 3, top // s, top // s - 1, rng.randint(0, top // s)):
            es |= {q * s + o for o in (-1, 0, 1)}
        for e in es:
            if 0 <= e <= top:
                assert lib.tree_row_of_draw(e, s) == e // s, (e, s)
