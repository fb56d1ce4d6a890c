"""Rows to their places in the stream, and the call's result to the host: by the compaction (numbers of rows where its workgroups
take more than four of them, end in a ragged one or leave the sums to a scan) and by the row coder itself, and calls that fail
in between.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import pcc_oracle as po
from paper_2212_01185_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def codec():
    from paper_2212_01185_amd import binding
    c = binding.Codec(synth.make_blob(0), 0)
    yield c
    c.close()


# 512 workgroups of four rows each; of eight (2,049 rows: the last workgroup has one); of a number that is no divisor of a row
# coder's 32; beyond 4,096 groups of 32, where a scan adds the groups up (131,105 rows: the last group has one)
@pytest.mark.parametrize("n,h,w", [(1, 2048, 1), (1, 2049, 5), (3, 2051, 2), (23, 1111, 1), (5, 26221, 1)])
def test_rows_and_offsets(codec, n, h, w):
    rng = np.random.default_rng(n * h + w)
    imgs = torch.from_numpy(rng.integers(0, 256, (n, h, w, 3), dtype=np.uint8)).cuda()
    stream = codec.pcc_encode(imgs)
    rows = n * h
    raw = stream.cpu().numpy()
    offsets = raw[32:32 + 8 * (rows + 1)].view(np.uint64).astype(np.int64)
    sizes = np.diff(offsets)
    assert offsets[0] == 0 and (sizes >= 16).all() and (sizes % 4 == 0).all()
    assert offsets[-1] == raw.size - 32 - 8 * (rows + 1)
    # every row's payload, from the intervals the pixel kernel made: the oracle's coder gives the same bytes
    sf = codec.pcc_copy_intervals(n, h, w).cpu().numpy().reshape(rows, 3 * w).astype(np.uint32)
    for r in sorted({0, 1, 31, 32, rows // 2, rows - 2, rows - 1} | set(rng.integers(0, rows, 40).tolist())):
        want = po.rans_encode(sf[r] & 0xFFFF, (sf[r] >> 16) + 1)
        at = 32 + 8 * (rows + 1) + offsets[r]
        assert raw[at:at + sizes[r]].tobytes() == want, r
    assert torch.equal(codec.pcc_decode(stream, n, h, w), imgs)


def test_a_call_that_fails_leaves_no_trace(codec):
    from paper_2212_01185_amd import binding
    rng = np.random.default_rng(5)
    imgs = torch.from_numpy(rng.integers(0, 256, (1, 70, 40, 3), dtype=np.uint8)).cuda()
    want = codec.pcc_encode(imgs).clone()
    for size in (want.numel() - 8, 32 + 8 * 71 + 64):
        for busy in (False, False, True):                # (the row coder runs beside the pixel kernel only where the stream is idle)
            out = torch.zeros(size // 8 * 8, dtype=torch.uint8, device="cuda")
            if not busy:
                torch.cuda.synchronize()
            with pytest.raises(binding.PccError) as e:
                codec.pcc_encode(imgs, out=out)
            assert e.value.code == binding.PCC_E_CAP
            torch.cuda.synchronize()
            assert torch.equal(codec.pcc_encode(imgs), want)


@pytest.mark.parametrize("env", [{"PCC_RANS_PATIENCE": "0"}, {"PCC_ENCODE_OVERLAP": "0"}])
def test_sequence_does_not_matter(codec, env, monkeypatch):
    from paper_2212_01185_amd import binding
    rng = np.random.default_rng(6)
    imgs = torch.from_numpy(rng.integers(0, 256, (2, 33, 300, 3), dtype=np.uint8)).cuda()
    want = codec.pcc_encode(imgs).clone()
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    other = binding.Codec(synth.make_blob(0), 0)
    try:
        for _ in range(3):
            assert torch.equal(other.pcc_encode(imgs), want)
    finally:
        other.close()


# The row coder places the rows of images of up to 1,024 columns itself where it has at most 96 groups of 32 rows: one group with
# a single row, with a row less than its waves, full and one row more; rows of fewer words than a wave's 256 and of several times
# as many; the most groups and one more; the widest image and one column more.  The compaction gives the same bytes.
@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 3, 40), (1, 32, 7), (1, 33, 300), (2, 37, 1024), (1, 34, 1025), (1, 3072, 9), (1, 3073, 9)])
def test_row_coder_places_rows_as_the_compaction_does(codec, n, h, w, monkeypatch):
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_ENCODE_OVERLAP", "0")
    other = binding.Codec(synth.make_blob(0), 0)
    rng = np.random.default_rng(3 * h + w)
    # noise (long rows) in the first half of the rows, an even grey (short ones) in the second
    imgs = rng.integers(0, 256, (n, h, w, 3), dtype=np.uint8)
    imgs[:, h // 2:] = 77
    imgs = torch.from_numpy(imgs).cuda()
    try:
        want = other.pcc_encode(imgs).clone()
        codec.pcc_set_profiling(True)
        for _ in range(3):
            out = torch.full((binding.pcc_stream_bound(n, h, w),), 0xA5, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()                                  # (an idle stream: beside the pixel kernel)
            got = codec.pcc_encode(imgs, out=out)
            ms = codec.pcc_last_timings()
            assert ms["encode_rans"] > 0 and (ms["encode_compact"] == 0) == (w <= 1024 and n * h <= 3072), ms
            assert torch.equal(got, want)
            assert bool((out[want.numel():] == 0xA5).all())           # nothing behind the stream
        small = (want.numel() - 4) // 8 * 8
        out.fill_(0xA5)
        torch.cuda.synchronize()
        with pytest.raises(binding.PccError) as e:                    # and nothing behind a buffer that is too small
            codec.pcc_encode(imgs, out=out[:small])
        assert e.value.code == binding.PCC_E_CAP and bool((out[small:] == 0xA5).all())
        assert torch.equal(codec.pcc_encode(imgs), want)
    finally:
        codec.pcc_set_profiling(False)
        other.close()


# A stream buffer that shares bytes with the images is written when all pixels have been read: by the compaction, behind the pixel
# kernel.  Stream's and image's first byte within one buffer: the same; the stream into the image's last bytes, and just behind them; the
# image into the stream's last possible byte, just behind it, and in its middle.
@pytest.mark.parametrize("h,w", [(40, 24), (512, 768)])
@pytest.mark.parametrize("where,shared", [("same", True), ("into end", True), ("behind", False), ("before", False), ("into front", True), ("inside", True)])
def test_stream_over_the_images(codec, h, w, where, shared):
    from paper_2212_01185_amd import binding
    imgs = torch.from_numpy(np.random.default_rng(h).integers(0, 256, (1, h, w, 3), dtype=np.uint8)).cuda()
    torch.cuda.synchronize()
    want = codec.pcc_encode(imgs).clone()
    size, bound = imgs.numel(), binding.pcc_stream_bound(1, h, w)
    assert size % 8 == 0
    img_at, stream_at = {"same": (0, 0), "into end": (0, size - 8), "behind": (0, size), "before": (bound, 0), "into front": (bound - 1, 0),
                         "inside": (bound // 3, 0)}[where]
    room = torch.empty(max(img_at + size, stream_at + bound), dtype=torch.uint8, device="cuda")
    view = room[img_at:img_at + size].view(1, h, w, 3)
    codec.pcc_set_profiling(True)
    try:
        for _ in range(3):
            view.copy_(imgs)
            torch.cuda.synchronize()
            got = codec.pcc_encode(view, out=room[stream_at:stream_at + bound])
            ms = codec.pcc_last_timings()
            assert torch.equal(got, want)
            assert ms["encode_rans"] > 0 and (ms["encode_compact"] > 0) == shared, ms
    finally:
        codec.pcc_set_profiling(False)


# The two ways in which a row coder's workgroup stands down while it places its rows: the sizes of those before it do not come (a
# limit of 0 polls: all but the first stand down at once), and one before it has stood down for want of a symbol (a few polls for
# those: some workgroups find theirs, some do not, differently in every call).  All rows are then coded again, the compaction places
# them, and the next call starts clean.
@pytest.mark.parametrize("symbols,sums", [(None, "0"), (None, "1")] + [(p, "100000") for p in ("0", "1", "2", "3", "5", "8", "12", "20")])
def test_workgroups_that_stand_down(codec, symbols, sums, monkeypatch):
    from paper_2212_01185_amd import binding
    if symbols is not None:
        monkeypatch.setenv("PCC_RANS_PATIENCE", symbols)
    monkeypatch.setenv("PCC_RANS_SUMS_PATIENCE", sums)
    other = binding.Codec(synth.make_blob(0), 0)
    rng = np.random.default_rng(9)
    try:
        other.pcc_set_profiling(True)
        for n, h, w in [(1, 32, 50), (1, 33, 7), (1, 512, 100), (3, 1000, 20), (1, 512, 768)]:
            imgs = torch.from_numpy(rng.integers(0, 256, (n, h, w, 3), dtype=np.uint8)).cuda()
            want = codec.pcc_encode(imgs).clone()
            out = torch.empty(binding.pcc_stream_bound(n, h, w), dtype=torch.uint8, device="cuda")
            for _ in range(6):
                out.fill_(0xA5)
                torch.cuda.synchronize()                 # (the row coder runs beside the pixel kernel only where the stream is idle)
                assert torch.equal(other.pcc_encode(imgs, out=out), want)
                assert bool((out[want.numel():] == 0xA5).all())
                placed_by_compaction = other.pcc_last_timings()["encode_compact"] > 0
                if sums == "0":
                    assert placed_by_compaction == (n * h > 32)
    finally:
        other.close()
