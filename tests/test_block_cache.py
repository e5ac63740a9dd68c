"""Host-only tests of the workspace block cache (runtime.cpp) against a mock
of the HIP runtime: whose blocks a stream is given."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_07096_amd", "csrc")
MB = 1 << 20
GB = 1 << 30
COUNTS = ["mallocs", "frees", "cross_waits", "unsafe_calls", "host_waits", "trims", "used"]


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    out = tmp_path_factory.mktemp("hipmock") / "libhipmock.so"
    # -Bsymbolic: the mock's own functions, also where the process has the real runtime loaded
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", "-Wno-unused-result", "-I", "/opt/rocm/include", "-I", CSRC,
                    os.path.join(CSRC, "runtime.cpp"), os.path.join(ROOT, "tests", "runtime_mock", "mock_hip.cpp"),
                    "-o", str(out)], check=True)
    return out


class Mock:
    def __init__(self, path):
        lib = C.CDLL(str(path))
        for f in ("mock_stream", "ws_new"):
            getattr(lib, f).restype = C.c_void_p
        lib.mock_count.restype = C.c_int64
        lib.mock_hammer.restype = C.c_int64
        lib.ws_new.argtypes = lib.ws_delete.argtypes = [C.c_void_p]
        lib.ws_alloc.argtypes = [C.c_void_p, C.c_size_t, C.POINTER(C.c_void_p)]
        lib.dev_alloc.argtypes = [C.c_size_t, C.POINTER(C.c_void_p)]
        lib.mock_capacity.argtypes = [C.c_size_t]
        lib.mock_capture.argtypes = [C.c_void_p, C.c_int]
        lib.mock_work.argtypes = lib.mock_finish.argtypes = [C.c_void_p]
        self.lib = lib

    def stream(self, dev=0):
        return self.lib.mock_stream(dev)

    def call(self, stream, *sizes, work=True, expect=0):
        """One library call: allocates the sizes, enqueues work, returns the blocks."""
        ws = self.lib.ws_new(stream)
        out = []
        for b in sizes:
            p = C.c_void_p()
            assert self.lib.ws_alloc(ws, b, C.byref(p)) == expect
            out.append(p.value)
        if work:
            self.lib.mock_work(stream)
        self.lib.ws_delete(ws)
        return out

    def __getattr__(self, name):
        if name in COUNTS:
            return self.lib.mock_count(COUNTS.index(name))
        return getattr(self.lib, "mock_" + name)


@pytest.fixture
def mock(so, tmp_path):
    # a copy per test: each loads a library with state of its own
    copy = tmp_path / "libhipmock.so"
    copy.write_bytes(so.read_bytes())
    return Mock(copy)


def test_same_stream_reuses_its_block(mock):
    s = mock.stream()
    blocks = {mock.call(s, 100 * MB)[0] for _ in range(10)}
    assert len(blocks) == 1 and mock.mallocs == 1 and mock.cross_waits == 0


def test_streams_do_not_wait_for_each_other(mock):
    a, b, c = mock.stream(), mock.stream(), mock.stream()
    for _ in range(4):  # nothing finishes: every stream keeps to its own blocks
        pa, pb, pc = (mock.call(s, 100 * MB, 1024)[0] for s in (a, b, c))
        assert len({pa, pb, pc}) == 3
    assert mock.cross_waits == 0
    assert mock.mallocs == 6  # two blocks a stream


def test_finished_block_serves_any_stream(mock):
    a, b = mock.stream(), mock.stream()
    p = mock.call(a, 100 * MB)
    mock.finish(a)
    assert mock.call(b, 90 * MB) == p
    assert mock.mallocs == 1 and mock.cross_waits == 0


def test_no_query_that_a_capture_elsewhere_forbids(mock):
    a, b, c = mock.stream(), mock.stream(), mock.stream()
    mock.call(a, 100 * MB)
    mock.capture(c, 1)
    mock.call(b, 100 * MB)  # looks at a's busy block
    mock.call(c, 100 * MB)  # the capturing stream owns its memory: no cached block
    assert mock.unsafe_calls == 0 and mock.mallocs == 3 and mock.cross_waits == 0
    mock.capture(c, 0)


def test_threads_never_share_a_block(mock):
    assert mock.hammer(8, 400) == 0
    assert mock.cross_waits == 0


def _idle(mock, s, count, size):
    """`count` idle blocks of `size` bytes, their work done."""
    ws = [mock.lib.ws_new(s) for _ in range(count)]
    for w in ws:
        assert mock.lib.ws_alloc(w, size, C.byref(C.c_void_p())) == 0
        mock.lib.mock_work(s)
    for w in ws:
        mock.lib.ws_delete(w)
    mock.finish(s)


@pytest.mark.parametrize("size", [900 * MB, 3 * GB])  # below and above what the cache keeps
def test_idle_blocks_are_given_back_when_a_request_fails(mock, size):
    s = mock.stream()
    mock.capacity(4 * GB)
    _idle(mock, s, 9, 200 * MB)
    assert mock.used >= 1800 * MB
    mock.capacity(size + 100 * MB)
    mock.call(s, size)
    assert mock.used <= size + 100 * MB and mock.trims >= 1


def test_idle_blocks_are_given_back_when_an_index_block_fails(mock):
    s = mock.stream()
    mock.capacity(2 * GB)
    _idle(mock, s, 8, 200 * MB)
    assert mock.lib.dev_alloc(1 * GB, C.byref(C.c_void_p())) == 0


def test_a_request_past_the_memory_still_fails(mock):
    s = mock.stream()
    mock.capacity(2 * GB)
    _idle(mock, s, 8, 200 * MB)
    nomem = 2  # STAG_E_NOMEM
    mock.call(s, 3 * GB, work=False, expect=nomem)
    assert mock.lib.dev_alloc(3 * GB, C.byref(C.c_void_p())) == nomem
    mock.call(s, 100 * MB)


def test_capturing_request_that_fails_leaves_the_cache_alone(mock):
    s, c = mock.stream(), mock.stream()
    mock.capacity(2 * GB)
    _idle(mock, s, 8, 200 * MB)
    mock.capture(c, 1)
    mock.call(c, 1 * GB, work=False, expect=2)
    assert mock.frees == 0 and mock.unsafe_calls == 0
    # on a stream that does not capture: nothing that would end the capture
    mock.call(s, 3 * GB // 2)
    assert mock.unsafe_calls == 0


def test_sizes_that_nobody_asks_for_make_room(mock):
    s = mock.stream()
    _idle(mock, s, 20, 100 * MB)  # 2000 MB idle, the limit is 2 GiB
    before = mock.mallocs
    for _ in range(10):
        mock.call(s, 300 * MB)
        mock.finish(s)
    assert mock.mallocs == before + 1  # kept after its first use
    assert mock.used <= 2 * GB


def test_blocks_at_work_are_not_evicted(mock):
    a, b = mock.stream(), mock.stream()
    ws = [mock.lib.ws_new(a) for _ in range(20)]
    for w in ws:
        assert mock.lib.ws_alloc(w, 100 * MB, C.byref(C.c_void_p())) == 0
    mock.lib.mock_work(a)
    for w in ws:
        mock.lib.ws_delete(w)
    mock.call(b, 300 * MB)  # goes back to the pool itself: all else is in use
    assert mock.cross_waits == 0 and mock.host_waits == 0 and mock.used == 2000 * MB


def test_blocks_stay_on_their_streams_device(mock):
    a, b = mock.stream(0), mock.stream(1)  # device 0 is current throughout
    pa = mock.call(a, 100 * MB)
    mock.finish(a)
    pb = mock.call(b, 100 * MB)
    mock.finish(b)
    assert pa != pb
    assert mock.call(a, 100 * MB) == pa and mock.call(b, 100 * MB) == pb
