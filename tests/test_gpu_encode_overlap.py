"""The row coder of a small encode runs on a stream of its codec's own, beside the pixel kernel on the caller's.  Streams share
the process's few hardware queues: with several codecs and callers' streams some pair shares one, and its two kernels run
one after the other.  Needs an MI355X."""
import time

import numpy as np
import pytest

from paper_2212_01185_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _log(msg):
    print(msg, flush=True)


def test_no_encode_waits_out_the_row_coders_patience(blob, monkeypatch):
    """With a patience of about 0.1 s, a row coder queued in front of the pixel kernel that it waits for would take that
    long.  Every pair of a codec and a caller's stream has to do without (a call takes tenths of a millisecond; the best of
    three counts, so that a busy host does not)."""
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_RANS_PATIENCE", "100000")
    codecs = [binding.Codec(blob, 0) for _ in range(8)]
    streams = [torch.cuda.default_stream()] + [torch.cuda.Stream() for _ in range(4)]
    # few rows (the row coder follows one pixel kernel) and many (it joins for a last part of the strips)
    shapes = [(1, 96, 128), (1, 1200, 100)]
    try:
        for n, h, w in shapes:
            imgs = torch.from_numpy(np.random.default_rng(95).integers(0, 256, (n, h, w, 3), dtype=np.uint8)).cuda()
            want = codecs[0].pcc_encode(imgs).clone()
            torch.cuda.synchronize()
            slowest = 0.0
            for s in streams:
                with torch.cuda.stream(s):
                    for c in codecs:
                        best = 1e9
                        for _ in range(3):
                            s.synchronize()
                            start = time.perf_counter()
                            got = c.pcc_encode(imgs)
                            best = min(best, time.perf_counter() - start)
                            if best < 0.02:
                                break
                        assert torch.equal(got, want)
                        slowest = max(slowest, best)
            _log("%dx%d: slowest of %d pairs %.2f ms" % (w, h, len(streams) * len(codecs), 1e3 * slowest))
            assert slowest < 0.02
    finally:
        for c in codecs:
            c.close()


def test_a_busy_null_stream_does_not_matter(blob):
    """A codec's first encode clears the buffer through which the row coder gets its symbols.  On the null stream, which other
    streams do not wait for, the clearing came behind whatever was queued there: after the pixel kernel, whose symbols it wiped."""
    from paper_2212_01185_amd import binding
    imgs = torch.from_numpy(np.random.default_rng(96).integers(0, 256, (1, 128, 128, 3), dtype=np.uint8)).cuda()
    known = binding.Codec(blob, 0)
    want = known.pcc_encode(imgs).clone()
    intervals = known.pcc_copy_intervals(1, 128, 128)
    known.close()
    out = torch.empty(binding.pcc_stream_bound(1, 128, 128), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        codec, s = binding.Codec(blob, 0), torch.cuda.Stream()
        try:
            torch.cuda.synchronize()
            torch.cuda._sleep(100_000_000)           # some 40 ms
            with torch.cuda.stream(s):
                got = codec.pcc_encode(imgs, out=out)
            torch.cuda.synchronize()
            assert torch.equal(got, want)
            assert torch.equal(codec.pcc_copy_intervals(1, 128, 128), intervals)
        finally:
            codec.close()
