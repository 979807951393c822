"""What a pull of the hand-off table gathers: whole and ragged chunks, more images than one launch takes, pieces that a
copy of their own has to move (off 16-byte alignment, pinned host memory).  Bytes must arrive as they were."""
import pytest

from parity_util import say

pytestmark = pytest.mark.gpu

CHUNK = 32768


@pytest.mark.parametrize("label,sizes,shift,pinned", [
    ("one byte", [1], 0, False),
    ("around 16 bytes and a chunk, off alignment after the first", [16, 17, CHUNK - 16, CHUNK, CHUNK + 16, 3 * CHUNK - 1, 15], 0, True),
    ("ragged last chunks", [CHUNK + 48, 5 * CHUNK + 32, 16, 2 * CHUNK - 16, CHUNK + 7], 0, True),
    ("sources off alignment", [4096, CHUNK + 64, 160], 2, True),
    ("more images than one launch takes", [16 * (1 + i % 37) + CHUNK * (i % 3) for i in range(300)], 0, True),
    ("one launch but for the pinned image", [64] * 128, 0, True),
    ("exactly one launch", [64] * 128, 0, False),
    ("one launch and one image", [64] * 129, 0, False),
])
def test_pull_moves_every_byte(label, sizes, shift, pinned):
    import torch

    import paper_2502_00937_amd as V

    say(f"case hand-off: {label}")
    g = torch.Generator().manual_seed(len(sizes))
    pieces = [torch.randint(0, 256, (n + shift,), dtype=torch.uint8, generator=g) for n in sizes]
    dev = [p.cuda() for p in pieces]
    host = pieces[0].pin_memory() if pinned else None  # one image in pinned host memory
    total = sum(sizes)
    dst = torch.zeros(total + 64, dtype=torch.uint8, device="cuda")
    h = V.TokenHandoff(0)
    h.expect(1, len(sizes))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for i in reversed(range(len(sizes))):
        src = host if host is not None and i == 0 else dev[i]
        h.publish(1, i, src.data_ptr() + shift, sizes[i], side.cuda_stream if i % 2 else torch.cuda.current_stream().cuda_stream)
    assert h.complete(1) == (True, total)
    assert h.pull(1, dst.data_ptr(), total, side.cuda_stream) == total
    torch.cuda.synchronize()
    want = torch.cat([p[shift:] for p in pieces])
    assert torch.equal(dst[:total].cpu(), want)
    assert int(dst[total:].max()) == 0  # nothing behind the request
    h.release(1)
    h.close()


@pytest.mark.parametrize("producer", ["own stream", "null stream behind a blocking stream", "blocking stream behind the null stream"])
def test_pull_waits_for_a_producer_at_work(producer):
    """The tokens are written late: by the publishing stream itself, or by a blocking stream whose work the null stream, which
    publishes them, comes after, or the other way round."""
    import ctypes

    import torch

    import paper_2502_00937_amd as V

    say(f"case hand-off of tokens still being written: {producer}")
    hip = ctypes.CDLL("libamdhip64.so")
    raw = ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(raw)) == 0  # a blocking stream
    work = torch.cuda.ExternalStream(raw.value)
    tokens = [torch.zeros(200000, dtype=torch.uint8, device="cuda") for _ in range(3)]
    dst = torch.zeros(600000, dtype=torch.uint8, device="cuda")
    consumer = torch.cuda.Stream()
    torch.cuda.synchronize()
    h = V.TokenHandoff(0)
    for rid in range(3):
        h.expect(rid, 3)
        with torch.cuda.stream(torch.cuda.default_stream() if producer.startswith("blocking") else work):
            torch.cuda._sleep(20_000_000)  # some milliseconds
            for i, t in enumerate(tokens):
                t.fill_(10 * rid + i + 1)
        for i, t in enumerate(tokens):
            h.publish(rid, i, t.data_ptr(), t.numel(), 0 if producer.startswith("null") else work.cuda_stream)
        h.pull(rid, dst.data_ptr(), dst.numel(), consumer.cuda_stream)
        consumer.synchronize()
        got = dst.view(3, -1).cpu()
        assert [(int(r.min()), int(r.max())) for r in got] == [(10 * rid + i + 1,) * 2 for i in range(3)]
        h.release(rid)
    h.close()
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(raw) == 0


@pytest.mark.parametrize("order", ["idle first", "at work first"])
def test_idle_and_busy_publishes_in_one_request(order):
    """Images with and without an event in one pull, more than a group's bytes of each."""
    import torch

    import paper_2502_00937_amd as V

    say(f"case hand-off of finished and unfinished images: {order}")
    n = 12 << 20
    idle, producer, consumer = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    tokens = [torch.full((n,), i + 1, dtype=torch.uint8, device="cuda") for i in range(6)]
    dst = torch.zeros(6 * n, dtype=torch.uint8, device="cuda")
    h = V.TokenHandoff(0)
    for rid in range(3):
        torch.cuda.synchronize()
        h.expect(rid, 6)
        late = range(2, 6) if order == "idle first" else range(0, 4)
        for i in range(6):
            if i == late[0]:
                with torch.cuda.stream(producer):
                    torch.cuda._sleep(20_000_000)
                    for k in late:
                        tokens[k].fill_(100 + 10 * rid + k)
            h.publish(rid, i, tokens[i].data_ptr(), n, producer.cuda_stream if i in late else idle.cuda_stream)
        h.pull(rid, dst.data_ptr(), dst.numel(), consumer.cuda_stream)
        consumer.synchronize()
        got = dst.view(6, n)
        assert [(int(r.min()), int(r.max())) for r in got] == [(100 + 10 * rid + i if i in late else i + 1,) * 2 for i in range(6)]
        h.release(rid)
    h.close()


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_a_capture_lives_through_publish_and_pull(mode):
    """Published and pulled on a stream under capture: the gather becomes part of the graph, and each replay moves what the
    sources hold then."""
    import torch

    import paper_2502_00937_amd as V

    say(f"case hand-off under capture, {mode}")
    tokens = [torch.zeros(CHUNK + 64, dtype=torch.uint8, device="cuda") for _ in range(3)]
    dst = torch.zeros(3 * (CHUNK + 64), dtype=torch.uint8, device="cuda")
    h = V.TokenHandoff(0)
    h.expect(1, 3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        s = torch.cuda.current_stream().cuda_stream
        for i, t in enumerate(tokens):
            h.publish(1, i, t.data_ptr(), t.numel(), s)
        h.pull(1, dst.data_ptr(), dst.numel(), s)
    for k in range(3):
        for i, t in enumerate(tokens):
            t.fill_(10 * k + i + 1)
        graph.replay()
        torch.cuda.synchronize()
        assert [(int(r.min()), int(r.max())) for r in dst.view(3, -1)] == [(10 * k + i + 1,) * 2 for i in range(3)]
    h.close()
