"""The host side of the one-shot calls without a GPU: how they stage their
descriptors on streams that are busy, capturing or of another device.  Each
case runs in a process of its own on tests/fake_hip.cpp, whose runtime calls
take the place of the real ones."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
A, B, C = 0x10, 0x20, 0x30  # streams


class Calls:
    """One-shot calls on n small neurons; tables and codes are never read."""

    def __init__(self, tt, fake):
        self.tt, self.L, self.fake = tt, tt.lib(), fake

    def desc(self, n):
        d = np.zeros(n, self.tt.NEURON_DTYPE)
        d["F"], d["b"], d["o"], d["w"][:, :2] = 2, 1, 1, 1
        return d, self.tt.layout(d)

    def enumerate(self, stream, n=16):
        d, total = self.desc(n)
        t = np.zeros(total, np.uint64)
        assert self.L.tt_enumerate(d.ctypes.data, n, t.ctypes.data, total, None, stream) == 0

    def pack(self, stream, n=16):
        d, total = self.desc(n)
        t = np.zeros(total, np.uint64)
        assert self.L.tt_pack(d.ctypes.data, n, t.ctypes.data, 4 * n, t.ctypes.data, total, stream) == 0

    def support(self, stream, n=16):
        d, total = self.desc(n)
        t = np.zeros(total, np.uint64)
        assert self.L.tt_support(d.ctypes.data, n, t.ctypes.data, total, t.ctypes.data, None, stream) == 0

    def noalloc(self, stream, n=16):
        d, total = self.desc(n)
        t = np.zeros(total, np.uint64)
        assert self.L.tt_enumerate_noalloc(d.ctypes.data, n, t.ctypes.data, total, None, stream) == 0

    def all(self, stream, n=16):
        for call in (self.enumerate, self.pack, self.support):
            call(stream, n)


def calls_while_another_stream_captures(c, fake):
    """A program records a graph on one stream and makes a call on another:
    the capture goes on, and the call is staged as ever."""
    c.all(A)
    fake.fake_capture(C)
    fake.fake_block(A)
    c.all(A)
    c.all(B)
    assert not fake.fake_invalidated()
    assert fake.fake_host_allocs() >= 4 and not fake.fake_graph_host_functions()


def calls_wait_for_no_other_stream(c, fake):
    """Calls for every buffer behind work that does not end, then calls on an
    idle stream: these never wait, no buffer that a queued call still reads is
    written again, and the buffers are bounded and used again later."""
    fake.fake_block(A)
    while fake.fake_host_allocs() == fake.fake_sources():
        c.pack(A)
        assert fake.fake_sources() < 100
    assert fake.fake_host_allocs() == 16
    # the last call found no buffer, could not wait for its stream's oldest, and copied from pageable memory
    waits = fake.fake_waits()
    read = [fake.fake_source(k) for k in range(fake.fake_sources())]
    assert waits <= 1 and len(set(read)) == 17
    for _ in range(20):
        c.all(B)
    assert fake.fake_waits() == waits and fake.fake_host_allocs() == 16
    assert not {fake.fake_source(k) for k in range(17, fake.fake_sources())} & set(read[:16])
    fake.fake_unblock(A)
    for _ in range(20):
        c.all(A)
    assert fake.fake_host_allocs() == 16 and fake.fake_waits() == waits


def a_larger_call_frees_no_buffer(c, fake):
    """A buffer that served a small call serves a large one as it is: freeing
    it to make a larger one would wait for every stream."""
    c.pack(B)
    fake.fake_block(A)
    c.pack(B, n=9000)  # 144 kB of records
    c.enumerate(B, n=16000)
    assert fake.fake_host_frees() == 0 and fake.fake_waits() == 0
    assert fake.fake_host_allocs() == 1


def a_buffer_of_unknown_state_is_not_used_again(c, fake):
    """Where the event behind a call cannot be recorded and the stream cannot
    be waited for, nobody knows when the call's buffer has been read."""
    fake.fake_block(A)
    fake.fake_fail_record(1)
    d, total = c.desc(16)
    t = np.zeros(total, np.uint64)
    assert c.L.tt_pack(d.ctypes.data, 16, t.ctypes.data, 64, t.ctypes.data, total, A) == c.tt.TT_EHIP
    for _ in range(20):
        c.pack(B)
    assert fake.fake_source(0) not in {fake.fake_source(k) for k in range(1, fake.fake_sources())}


def a_stream_of_another_device(c, fake):
    """A call on a stream of a device that is not the current one succeeds."""
    fake.fake_stream_device(B, 1)
    c.all(A)
    c.all(B)
    c.all(A)


def a_captured_copy_lives_as_long_as_its_graph(c, fake):
    """A call recorded into a graph: replays read the call's own copy of its
    descriptors, which nothing frees before the graph is destroyed."""
    for call in (c.noalloc, c.enumerate, c.pack, c.support):
        fake.fake_capture(A)
        call(A)
        fake.fake_capture(None)
        assert fake.fake_graph_host_functions() == 0 and fake.fake_retained() == 1
        sums = []
        for _ in range(3):
            sums.append(fake.fake_replay())
            c.all(B, 100)  # host memory that was free by now is written
        assert sums[0] > 0 and sums == sums[:1] * 3
        fake.fake_destroy_graph()
    assert not fake.fake_invalidated()


CASES = [calls_while_another_stream_captures, calls_wait_for_no_other_stream, a_larger_call_frees_no_buffer,
         a_buffer_of_unknown_state_is_not_used_again, a_stream_of_another_device,
         a_captured_copy_lives_as_long_as_its_graph]


@pytest.fixture(scope="module")
def fake_so(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "fake_hip.cpp")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", src, "-o", out])
    return out


@pytest.mark.parametrize("case", [f.__name__ for f in CASES])
def test_staging(case, fake_so):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), case, fake_so], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    stand_in = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)  # first, so that libtt.so finds its symbols here
    for name in ("fake_block", "fake_unblock", "fake_capture"):
        getattr(stand_in, name).argtypes = [ctypes.c_void_p]
    stand_in.fake_stream_device.argtypes = [ctypes.c_void_p, ctypes.c_int]
    stand_in.fake_source.restype = ctypes.c_void_p
    stand_in.fake_replay.restype = ctypes.c_long
    sys.path.insert(0, ROOT)
    import paper_2502_08673_amd as package

    {f.__name__: f for f in CASES}[sys.argv[1]](Calls(package, stand_in), stand_in)
