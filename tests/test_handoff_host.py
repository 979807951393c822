"""The hand-off table's host side, built against a small HIP runtime on the host (tests/host_hip): what its calls accept, what
they wait for and where the bytes arrive, with two devices and with producers that finish when the test says so."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.environ.get("HOST_CLANG", "/opt/rocm/llvm/bin/clang++")  # the kernel's vector types are clang's


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("handoff") / "libhandoff_host.so")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O2", "-fPIC", "-shared", "-I", os.path.join(HERE, "host_hip"),
                    os.path.join(HERE, "host_hip", "handoff_host.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.host_alloc.restype = lib.host_stream.restype = C.c_void_p
    lib.host_alloc.argtypes = [C.c_int, C.c_size_t]
    lib.host_work.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_size_t]
    lib.host_capture.argtypes = [C.c_void_p, C.c_int]
    lib.host_captured.argtypes = [C.c_void_p, C.POINTER(C.c_int)]
    lib.host_error.restype = C.c_char_p
    lib.vit_handoff_create.argtypes = [C.c_int, C.POINTER(C.c_void_p)]
    lib.vit_handoff_destroy.argtypes = [C.c_void_p]
    lib.vit_handoff_expect.argtypes = [C.c_void_p, C.c_int64, C.c_int32]
    lib.vit_handoff_publish.argtypes = [C.c_void_p, C.c_int64, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]
    lib.vit_handoff_pull.argtypes = [C.c_void_p, C.c_int64, C.c_void_p, C.c_size_t, C.c_void_p, C.POINTER(C.c_size_t)]
    lib.vit_handoff_release.argtypes = [C.c_void_p, C.c_int64]
    return lib


class Table:
    """A table on device 0, a request of the given images (each filled with its own bytes) and a destination."""

    def __init__(self, lib, sizes, dst_device=0):
        self.lib, self.sizes = lib, sizes
        self.h = C.c_void_p()
        assert lib.vit_handoff_create(0, C.byref(self.h)) == 0
        assert lib.vit_handoff_expect(self.h, 1, len(sizes)) == 0
        self.src = [lib.host_alloc(0, n) for n in sizes]
        self.dst = lib.host_alloc(dst_device, sum(sizes))
        self.want = np.random.default_rng(len(sizes)).integers(1, 256, sum(sizes), dtype=np.uint8)
        at = 0
        for p, n in zip(self.src, sizes):
            C.memmove(p, self.want[at:].ctypes.data, n)
            at += n

    def publish(self, i, stream, ptr=None):
        return self.lib.vit_handoff_publish(self.h, 1, i, ptr or self.src[i], self.sizes[i], stream)

    def pull(self, stream, dst=None):
        n = C.c_size_t()
        rc = self.lib.vit_handoff_pull(self.h, 1, dst or self.dst, sum(self.sizes), stream, C.byref(n))
        assert rc != 0 or n.value == sum(self.sizes)
        return rc

    def got(self, dst=None):
        return np.ctypeslib.as_array((C.c_uint8 * sum(self.sizes)).from_address(dst or self.dst)).copy()

    def image(self, i):
        at = sum(self.sizes[:i])
        return slice(at, at + self.sizes[i])

    def counts(self):
        out = (C.c_int * 4)()
        self.lib.host_counts(out)
        return dict(zip(("launches", "copies", "waits", "events"), out))


CHUNK = 32768


@pytest.mark.parametrize("sizes", [[1], [16, 17, CHUNK - 16, CHUNK, CHUNK + 16, 3 * CHUNK - 1, 15], [64] * 128, [64] * 129])
def test_every_byte_arrives(lib, sizes):
    t = Table(lib, sizes)
    t.counts()
    consumer = lib.host_stream(0, 0)
    for i in range(len(sizes)):
        assert t.publish(i, None) == 0
    assert t.pull(consumer) == 0
    lib.host_pump()
    assert np.array_equal(t.got(), t.want)
    if len(set(sizes)) == 1 and len(sizes) > 1:
        c = t.counts()
        assert (c["launches"], c["copies"]) == (-(-len(sizes) // 128), 0)
    lib.vit_handoff_destroy(t.h)


@pytest.mark.parametrize("busy", [False, True])
def test_a_stream_of_another_device_is_refused(lib, busy):
    """The table's events cannot be recorded on it: refused whether or not that stream has work left."""
    t = Table(lib, [4096])
    foreign = lib.host_stream(1, 0)
    if busy:
        lib.host_work(foreign, lib.host_alloc(1, 64), 1, 64)
    assert t.publish(0, foreign) == -4, lib.host_error()
    # nothing of the refused call stays behind: the image can still be published, and its stream is not taken to be at work
    t.counts()
    own = lib.host_stream(0, 0)
    assert t.publish(0, own) == 0
    assert t.counts()["events"] == 0
    lib.vit_handoff_destroy(t.h)


def test_a_blocking_stream_behind_the_null_stream_is_waited_for(lib):
    """An event recorded on an idle blocking stream comes after the work that the null stream was given before it; a query
    of that stream says that it is idle."""
    t = Table(lib, [4096])
    blocking, consumer = lib.host_stream(0, 1), lib.host_stream(0, 0)
    late = lib.host_work(None, t.src[0], 7, 4096)  # the tokens are still being written, on the null stream
    assert t.publish(0, blocking) == 0
    assert t.pull(consumer) == 0
    lib.host_pump()
    assert not t.got().any()
    lib.host_end_work(late)
    assert (t.got() == 7).all()
    lib.vit_handoff_destroy(t.h)


def test_a_stream_that_waits_for_nobody_needs_no_event(lib):
    """A non-blocking stream does not come after the null stream: idle is idle."""
    t = Table(lib, [4096])
    late = lib.host_work(None, lib.host_alloc(0, 64), 7, 64)
    t.counts()
    assert t.publish(0, lib.host_stream(0, 0)) == 0
    assert t.counts()["events"] == 0
    lib.host_end_work(late)
    lib.vit_handoff_destroy(t.h)


@pytest.mark.parametrize("shift", [2 * CHUNK, 3 * CHUNK, 5 * CHUNK])
def test_a_destination_over_the_sources_is_filled_in_image_order(lib, shift):
    """A request closed up towards the front of its own buffer: an image's place may be where an earlier image lay, which has
    been moved by then."""
    sizes = [2 * CHUNK] * 4
    t = Table(lib, sizes)
    step = 2 * CHUNK + shift
    buf = lib.host_alloc(0, shift + 4 * step)
    consumer = lib.host_stream(0, 0)
    for i in range(4):
        C.memmove(buf + shift + i * step, t.src[i], sizes[i])
        assert t.publish(i, None, buf + shift + i * step) == 0
    assert t.pull(consumer, buf) == 0
    lib.host_pump()
    assert np.array_equal(t.got(buf), t.want)
    lib.vit_handoff_destroy(t.h)


def test_tokens_already_in_place_are_gathered(lib):
    """A source that is its own destination meets nobody else's."""
    t = Table(lib, [2 * CHUNK] * 4)
    C.memmove(t.dst, t.want.ctypes.data, t.want.size)
    at = [t.dst + 2 * CHUNK * i for i in range(4)]
    t.counts()
    for i in range(4):
        assert t.publish(i, None, at[i] if i % 2 else None) == 0
    assert t.pull(lib.host_stream(0, 0)) == 0
    lib.host_pump()
    assert np.array_equal(t.got(), t.want) and t.counts()["copies"] == 0
    lib.vit_handoff_destroy(t.h)


@pytest.mark.parametrize("earlier", ["finished before", "own launch before"])
def test_finished_images_do_not_wait_for_the_last_one(lib, earlier):
    """All but the last image are there when the consumer pulls, or come from an earlier launch: they are moved while the
    last one is still being made."""
    n, size = 10, 5 * (1 << 20)
    t = Table(lib, [size] * n)
    producer, consumer = lib.host_stream(0, 0), lib.host_stream(0, 0)
    scratch = lib.host_alloc(0, 64)
    first = lib.host_work(producer, scratch, 1, 64) if earlier == "own launch before" else None
    for i in range(n - 1):
        assert t.publish(i, producer) == 0
    last = lib.host_work(producer, t.src[n - 1], 7, size)
    assert t.publish(n - 1, producer) == 0
    t.counts()
    assert t.pull(consumer) == 0
    assert t.counts()["launches"] < n  # not one launch per image
    lib.host_pump()
    if first is not None:
        assert not t.got().any()
        lib.host_end_work(first)
    got = t.got()
    there = [np.array_equal(got[t.image(i)], t.want[t.image(i)]) for i in range(n - 1)]
    assert sum(there) >= n - 1 - (3 if first is not None else 0), there  # images of an unfinished event go in groups
    assert not got[t.image(n - 1)].any()
    lib.host_end_work(last)
    got = t.got()
    assert np.array_equal(got[:-size], t.want[:-size]) and (got[-size:] == 7).all()
    lib.vit_handoff_destroy(t.h)


@pytest.mark.parametrize("order", ["idle first", "at work first"])
def test_idle_and_busy_publishes_in_one_request(lib, order):
    t = Table(lib, [CHUNK + 16] * 3)
    idle, producer, consumer = lib.host_stream(0, 0), lib.host_stream(0, 0), lib.host_stream(0, 0)
    late = lib.host_work(producer, t.src[1], 9, CHUNK + 16)
    for i, s in ((0, idle), (1, producer), (2, idle)) if order == "idle first" else ((1, producer), (0, idle), (2, idle)):
        assert t.publish(i, s) == 0
    assert t.pull(consumer) == 0
    lib.host_pump()
    assert not t.got()[t.image(1)].any()
    lib.host_end_work(late)
    got = t.got()
    assert (got[t.image(1)] == 9).all() and all(np.array_equal(got[t.image(i)], t.want[t.image(i)]) for i in (0, 2))
    lib.vit_handoff_destroy(t.h)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("who", ["producer", "consumer", "another"])
def test_a_capture_lives_through_publish_and_pull(lib, who, mode):
    """Neither call asks a question that would end a capture, of the producer's stream, the consumer's or a third one."""
    t = Table(lib, [4096] * 3)
    s = {k: lib.host_stream(0, 0) for k in ("producer", "consumer", "another", "busy")}
    late = lib.host_work(s["busy"], t.src[2], 5, 4096)
    lib.host_capture(s[who], mode)
    assert [t.publish(0, s["producer"]), t.publish(1, s["producer"]), t.publish(2, s["busy"])] == [0, 0, 0]
    assert t.pull(s["consumer"]) == 0
    recorded = C.c_int()
    assert lib.host_captured(s[who], C.byref(recorded)) == 1
    assert (recorded.value > 0) == (who != "another")
    lib.host_capture(s[who], -1)
    lib.host_end_work(late)
    if who != "consumer":
        assert (t.got()[t.image(2)] == 5).all()
    lib.vit_handoff_destroy(t.h)
