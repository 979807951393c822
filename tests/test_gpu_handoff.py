"""What a pull of the hand-off table gathers: whole and ragged chunks, more images than one launch takes, pieces that a
copy of their own has to move (off 16-byte alignment, pinned host memory).  Bytes must arrive as they were."""
import pytest

from parity_util import say

pytestmark = pytest.mark.gpu

CHUNK = 32768


@pytest.mark.parametrize("label,sizes,shift", [
    ("one byte", [1], 0),
    ("around 16 bytes and a chunk, off alignment after the first", [16, 17, CHUNK - 16, CHUNK, CHUNK + 16, 3 * CHUNK - 1, 15], 0),
    ("ragged last chunks", [CHUNK + 48, 5 * CHUNK + 32, 16, 2 * CHUNK - 16, CHUNK + 7], 0),
    ("sources off alignment", [4096, CHUNK + 64, 160], 2),
    ("more images than one launch takes", [16 * (1 + i % 37) + CHUNK * (i % 3) for i in range(300)], 0),
    ("exactly one launch", [64] * 128, 0),
])
def test_pull_moves_every_byte(label, sizes, shift):
    import torch

    import paper_2502_00937_amd as V

    say(f"case hand-off: {label}")
    g = torch.Generator().manual_seed(len(sizes))
    pieces = [torch.randint(0, 256, (n + shift,), dtype=torch.uint8, generator=g) for n in sizes]
    dev = [p.cuda() for p in pieces]
    host = pieces[0].pin_memory() if len(sizes) > 2 else None  # one image in pinned host memory
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
