"""Host-only tests of what the chunks of a served CKNS request may take for the
pairs that its queries meet: inside the budget, and no request that its other
bytes admit is refused."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_07096_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("allowance") / "liballowance.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-I", CSRC,
                    os.path.join(ROOT, "tests", "serve_mock", "allowance.cpp"), "-o", str(out)], check=True)
    lib = C.CDLL(str(out))
    lib.at_once.restype = C.c_int64
    lib.at_once.argtypes = [C.c_int64, C.c_int64, C.c_int32]
    lib.allowance.restype = C.c_uint64
    lib.allowance.argtypes = [C.c_uint64, C.c_int32, C.c_int64, C.c_int64, C.c_uint64, C.c_uint64]
    return lib


def test_allowance_stays_inside_the_budget(lib):
    rng = random.Random(5)
    for _ in range(2000):
        budget, streams = rng.randint(1, 1 << 35), rng.randint(1, 16)
        chunk, m = rng.choice([512, 4096, 1 << 20]), rng.randint(1, 1 << 20)
        base, need = rng.randint(1, 1 << 33), rng.randint(0, 1 << 32)
        a = lib.allowance(budget, streams, chunk, m, base, need)
        k = lib.at_once(m, chunk, streams)
        assert 1 <= k <= streams and a <= need
        if base <= budget:
            assert base + k * a <= budget  # admitted, as by its base alone
        else:
            assert a == 0
        assert k * a <= budget // 2  # other requests keep their part


def test_allowance_is_all_that_is_needed_where_the_budget_has_it(lib):
    gb = 1 << 30
    assert lib.allowance(8 * gb, 4, 4096, 100000, 300 << 20, gb) == gb
    assert lib.allowance(8 * gb, 4, 4096, 256, 65 << 20, 33 << 20) == 33 << 20
    assert lib.allowance(8 * gb, 16, 4096, 100000, 300 << 20, gb) == gb // 4
