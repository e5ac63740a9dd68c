"""Host-only tests of the memory that CKNS queries take (lsh.hip on a mock of
the HIP runtime, kernels not run): what fits, what is done in slices and what
fails."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_07096_amd", "csrc")
MOCK = os.path.join(ROOT, "tests", "runtime_mock")
GB = 1 << 30
OK, NOMEM, UNSUPPORTED = 0, 2, 4


def build(out, unit):
    """The mocked library around one test unit that includes a HIP source."""
    flags = ["-O1", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC, "-I", MOCK]
    obj = str(out / "unit.o")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", *flags, "-c",
                    os.path.join(MOCK, unit), "-o", obj], check=True)
    und = subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout
    fat = [s.split()[-1] for s in und.splitlines() if "__hip_fatbin" in s]
    lib = str(out / "libmock.so")
    subprocess.run(["g++", "-shared", "-pthread", "-Wl,-Bsymbolic", "-Wno-unused-result", *flags, obj,
                    os.path.join(CSRC, "runtime.cpp"), os.path.join(MOCK, "mock_hip.cpp"),
                    os.path.join(MOCK, "mock_launch.cpp"), *[f"-Wl,--defsym={f}=mock_fatbin" for f in fat],
                    "-o", lib], check=True)
    return lib


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return build(tmp_path_factory.mktemp("lshmock"), "lsh_host.cpp")


@pytest.fixture
def lib(so, tmp_path):
    copy = tmp_path / "libmock.so"  # a state of its own for every test
    shutil.copy(so, copy)
    lib = C.CDLL(str(copy))
    for f in ("mock_stream", "lsh_index"):
        getattr(lib, f).restype = C.c_void_p
    for f in ("mock_count", "lsh_combined", "launch_threads", "launch_count"):
        getattr(lib, f).restype = C.c_int64
    lib.mock_capacity.argtypes = [C.c_size_t]
    lib.lsh_index.argtypes = [C.c_int] * 5 + [C.c_int64]
    lib.lsh_free.argtypes = [C.c_void_p]
    lib.lsh_query.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_int64, C.c_uint64]
    lib.lsh_members.argtypes = lib.lsh_pairs.argtypes = [C.c_void_p, C.c_int64]
    lib.lsh_pairs.restype = C.c_uint64
    lib.lsh_combined.argtypes = [C.c_void_p, C.c_void_p, C.c_int64]
    lib.launch_count.argtypes = [C.c_char_p]
    lib.lsh_dense.argtypes = [C.c_void_p, C.c_int]
    lib.lsh_sample.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_int]
    lib.lsh_bucket_tasks.restype = C.c_uint32
    lib.lsh_bucket_tasks.argtypes = [C.c_uint32, C.c_uint32]
    return lib


@pytest.fixture
def stream(lib):
    return lib.mock_stream(0)


def combined(lib):
    """The query ranges whose results were combined, in order."""
    cap = 100000
    q0, count = (C.c_int64 * cap)(), (C.c_int64 * cap)()
    k = lib.lsh_combined(q0, count, cap)
    return [(q0[i], count[i]) for i in range(k)]


def covers(lib, m):
    at = 0
    for q0, c in combined(lib):
        assert q0 == at and c > 0
        at += c
    return at == m


def test_join_in_one_slice(lib, stream):
    idx = lib.lsh_index(64, 1, 17, 4, 6, 1 << 20)
    assert lib.lsh_query(idx, stream, 4096, 100, 0) == OK
    assert combined(lib) == [(0, 4096)]
    lib.lsh_free(idx)


@pytest.mark.parametrize("tasks", [3000, 40000, 1000000])  # a query: 1e7, 1.6e8 and 4e9 in a batch
def test_join_with_many_tasks(lib, stream, tasks):
    # wide kernels, where most points share a bucket: more tasks than a launch
    # or the memory takes are done in slices of the queries
    idx = lib.lsh_index(64, 1, 17, 4, 6, 1 << 20)
    lib.mock_capacity(20 * GB)
    assert lib.lsh_query(idx, stream, 4096, tasks, 0) == OK
    assert covers(lib, 4096)
    assert lib.launch_threads() < 1 << 32
    lib.lsh_free(idx)


def test_join_in_little_memory(lib, stream):
    idx = lib.lsh_index(64, 1, 17, 4, 6, 1 << 20)
    lib.mock_capacity(1 * GB)
    assert lib.lsh_query(idx, stream, 4096, 1000, 0) == OK  # 2.3 GB of tasks at once
    assert covers(lib, 4096)
    lib.mock_capacity(32 << 20)  # not even a block
    assert lib.lsh_query(idx, stream, 100000, 1000, 0) == NOMEM
    lib.lsh_free(idx)


def test_tasks_of_a_bucket(lib):
    for nq, nm in [(0, 5), (5, 0), (1, 1), (64, 128), (65, 129), (1 << 27, 1 << 20), (1 << 27, (1 << 31) - 1)]:
        assert lib.lsh_bucket_tasks(nq, nm) == min(-(-nq // 64) * -(-nm // 128), (1 << 32) - 1)


def test_join_of_a_query_past_the_launch(lib, stream):
    idx = lib.lsh_index(64, 1, 17, 4, 6, 1 << 20)
    assert lib.lsh_query(idx, stream, 64, 1 << 27, 0) == UNSUPPORTED
    lib.lsh_free(idx)


@pytest.mark.parametrize("capacity,pairs", [(8192, True), (1000, True), (600, True), (220, True), (90, False)])
@pytest.mark.parametrize("draws", [0, 5])
def test_dense_levels_in_little_memory(lib, stream, capacity, pairs, draws):
    # 38,400 dense columns: 1.4 GB of pairs for 4,096 queries at once (3.3 with
    # draws), 44 MB (103) for 128, and twice 64 MB of small buffers; without even
    # these every level is walked
    idx = lib.lsh_index(200, 1, 17, 4, 6, 1 << 20)
    lib.lsh_dense(idx, 300)
    if draws:
        capacity *= 2
    lib.mock_capacity(capacity << 20)
    if draws:
        assert lib.lsh_sample(idx, stream, 4096, draws) == OK
    else:
        assert lib.lsh_query(idx, stream, 4096, 0, 0) == OK
    assert (lib.launch_count(b"dense_pairs") > 0) == pairs
    assert lib.launch_count(b"dense_pairs") == lib.launch_count(b"dense_terms")
    assert lib.launch_count(b"probe_queries") > 0
    lib.lsh_free(idx)


PEAK = 7


@pytest.mark.parametrize("limit", [60 << 20, 200 << 20, 500 << 20])
def test_dense_pairs_within_a_limit(lib, stream, limit):
    idx = lib.lsh_index(200, 1, 17, 4, 6, 1 << 20)
    lib.lsh_dense(idx, 300)
    assert lib.lsh_pairs(idx, 100) == 128 * 38400 * 9 and lib.lsh_pairs(idx, 1 << 20) == 1 << 30
    assert lib.lsh_query(idx, stream, 4096, 0, limit) == OK
    assert lib.launch_count(b"dense_pairs") > 0
    assert lib.mock_count(PEAK) <= limit + (2 * 64 << 20)  # and the blocks of the small buffers
    lib.lsh_free(idx)


@pytest.mark.parametrize("limit", [1 << 20, 100 << 20])
def test_join_tasks_within_a_limit(lib, stream, limit):
    idx = lib.lsh_index(64, 1, 17, 4, 6, 1 << 16)
    assert lib.lsh_query(idx, stream, 4096, 1000, limit) == OK
    assert covers(lib, 4096)
    assert lib.mock_count(PEAK) <= limit + (2 * 64 << 20)
    lib.lsh_free(idx)


def test_pair_bytes_bound_the_tasks_of_a_join(lib):
    rng = random.Random(3)
    for _ in range(200):
        m, members, buckets = rng.randint(1, 5000), rng.randint(1, 20000), rng.choice([1, 2, 10, 300])
        nq, nm = [0] * buckets, [0] * buckets
        for _ in range(m):
            nq[min(rng.randrange(buckets), rng.randrange(buckets))] += 1
        for _ in range(members):
            nm[min(rng.randrange(buckets), rng.randrange(buckets))] += 1
        idx = lib.lsh_index(64, 1, 1, 1, 6, 1 << 16)
        lib.lsh_members(idx, members)
        tasks = sum(lib.lsh_bucket_tasks(a, b) for a, b in zip(nq, nm))
        assert tasks * 552 <= lib.lsh_pairs(idx, m)
        lib.lsh_free(idx)
