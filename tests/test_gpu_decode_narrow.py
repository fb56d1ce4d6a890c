"""The decoder with bands of eight rows: heights around whole bands of 8 and of 16 rows, widths from one pixel on, networks whose two
halves of the components are equal in number and not, several images, and the limit of the static scratch.  Needs an MI355X."""
import threading
import time

import numpy as np
import pytest

from paper_2212_01185_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NARROW = {"workload": (synth.DEFAULT_DIMS, {}), "paper": (synth.PAPER_DIMS, dict(k=3, nbhd=12, delay=3, act=synth.ACT_LEAKY))}
NARROW.update({name: (synth.ablation_dims(*shape), dict(k=shape[0], nbhd=12, delay=3, act=synth.ACT_LEAKY)) for name, shape in synth.ABLATION_SHAPES.items()})
BLOBS = {"workload": synth.make_blob, "paper": synth.make_paper_blob, "diagonal": synth.make_diagonal_blob}
BLOBS.update({name: lambda seed, name=name: synth.make_ablation_blob(*synth.ABLATION_SHAPES[name], seed=seed) for name in synth.ABLATION_SHAPES})
SIZES = [(1, 1, 1), (2, 7, 5), (1, 8, 33), (3, 9, 2), (1, 15, 40), (1, 16, 3), (2, 17, 18), (1, 23, 1), (5, 24, 31), (1, 25, 64), (1, 33, 17)]


@pytest.mark.parametrize("launch", ["0", "3"])
@pytest.mark.parametrize("net", sorted(BLOBS))
def test_bands_of_eight_rows_decode_exactly(net, launch, monkeypatch):
    """Chosen by the rule and forced: the images exactly."""
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_DECODE_VARIANT", launch)
    codec = binding.Codec(BLOBS[net](0), 0)
    rng = np.random.default_rng(11)
    try:
        for n, h, w in SIZES:
            print("%s %dx%dx%d" % (net, n, h, w), flush=True)
            imgs = torch.from_numpy(rng.integers(0, 256, (n, h, w, 3), dtype=np.uint8)).cuda()
            stream = codec.pcc_encode(imgs)
            assert torch.equal(codec.pcc_decode(stream, n, h, w), imgs)
            out = torch.zeros_like(imgs)
            assert torch.equal(codec.pcc_decode_static(stream, n, h, w, out), imgs)
    finally:
        codec.close()


@pytest.mark.parametrize("launch", ["0", "3"])
def test_static_scratch_too_small_for_twice_the_bands(launch, monkeypatch):
    """270 bands of eight rows of 4096 pixels would need 8.4 MiB of the 8 MiB, the 135 bands of 16 rows fit: accepted as ever."""
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_DECODE_VARIANT", launch)
    h, w = 2160, 4096
    assert binding.load().pcc_decode_static_scratch_bytes(1, h, w) <= 8 << 20 < 2 * 8 * 135 * w
    imgs = torch.from_numpy(synth.make_image(5, synth.ImageSpec(w, h, 12, 8.0, 64.0))).cuda()[None]
    codec = binding.Codec(synth.make_blob(0), 0)
    try:
        stream = codec.pcc_encode(imgs)
        assert torch.equal(codec.pcc_decode_static(stream, 1, h, w, torch.zeros_like(imgs)), imgs)
    finally:
        codec.close()


@pytest.mark.parametrize("net", sorted(NARROW))
def test_a_band_that_gives_up_ends_the_call(net, monkeypatch):
    """With the limit of a band's polls set to zero from the host the call returns an error, and the next one works: for jobs of
    more bands than the chip holds at once and of a few, with the flag read in B's search (the workload's network) and in the next
    step's head (no layer leaves a wave spare time)."""
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_DECODE_VARIANT", "3")
    good = binding.Codec(BLOBS[net](0), 0)
    monkeypatch.setenv("PCC_DECODE_SPIN_LIMIT", "0")
    hasty = binding.Codec(BLOBS[net](0), 0)
    try:
        imgs = torch.from_numpy(np.random.default_rng(79).integers(0, 256, (120, 40, 24, 3), dtype=np.uint8)).cuda()       # 600 bands
        for n in (120, 1):
            print("%s: decode without patience, %d images" % (net, n), flush=True)
            stream = good.pcc_encode(imgs[:n])
            for decode in (hasty.pcc_decode, lambda *a: hasty.pcc_decode_static(*a, torch.zeros_like(imgs[:n]))):
                with pytest.raises(binding.PccError) as e:
                    decode(stream, n, 40, 24)
                assert e.value.code == binding.PCC_E_INTERNAL
            assert torch.equal(good.pcc_decode(stream, n, 40, 24), imgs[:n])
    finally:
        good.close()
        hasty.close()


@pytest.mark.parametrize("net", sorted(NARROW))
def test_mixture_sums_that_are_not_numbers(net, monkeypatch):
    """A logit that is infinite or NaN makes the softmax and with it a channel's mixture sums NaN, which count as 1.  The second
    half of a pixel's lanes goes on with the first half's sum: logits of either half, in each channel."""
    from paper_2212_01185_amd import binding
    monkeypatch.setenv("PCC_DECODE_VARIANT", "3")
    dims, header = NARROW[net]
    k = header.get("k", 5)
    imgs = torch.from_numpy(np.random.default_rng(83).integers(0, 256, (2, 19, 24, 3), dtype=np.uint8)).cuda()
    for channel, component, value in [(0, 0, np.inf), (0, k - 1, np.nan), (1, k - 1, np.inf), (2, 0, np.nan), (2, k - 1, np.inf)]:
        layers = [[w, b.copy()] for w, b in synth.make_weights(0, dims)]
        layers[-1][1][3 * k * channel + component] = value
        codec = binding.Codec(synth.pack_blob(layers, **header), 0)
        print("%s: channel %d, component %d: %s" % (net, channel, component, value), flush=True)
        try:
            params, _ = codec.pcc_encode_probs(imgs)
            assert not torch.isfinite(params[..., 3 * k * channel + component]).any()
            stream = codec.pcc_encode(imgs)
            assert torch.equal(codec.pcc_decode(stream, 2, 19, 24), imgs)
        finally:
            codec.close()


@pytest.mark.parametrize("h, w, threads", [(2160, 4096, 3), (217, 333, 4)])
def test_decodes_that_run_at_once_share_the_chip(h, w, threads, monkeypatch):
    """Several threads decode, each with a codec and a stream of its own.  Bands of eight rows hold twice the places: where that
    many such jobs fill the chip they would wait for each other (three of 4096x2160: 1.4 times as long as with bands of
    16 rows), so the rule leaves them out.  Both ways take the same streams, others each time (two may share a hardware queue)."""
    from paper_2212_01185_amd import binding
    one = torch.from_numpy(synth.make_image(7, synth.ImageSpec(w, h, 12, 8.0, 64.0))).cuda()[None]
    codecs = {}
    for variant in ("1", "0"):
        monkeypatch.setenv("PCC_DECODE_VARIANT", variant)
        codecs[variant] = [binding.Codec(synth.make_blob(0), 0) for _ in range(threads)]
    outs = [torch.empty_like(one) for _ in range(threads)]
    ratios = []
    try:
        stream = codecs["0"][0].pcc_encode(one)
        for cs in codecs.values():
            for c, out in zip(cs, outs):
                c.pcc_decode(stream, 1, h, w, out=out)
        for _ in range(5):
            streams, seconds = [torch.cuda.Stream() for _ in outs], {}
            for variant, cs in codecs.items():
                for out in outs:
                    out.zero_()
                torch.cuda.synchronize()
                wrong = []

                def work(c, s, out):
                    with torch.cuda.stream(s):
                        try:
                            for _ in range(4):
                                c.pcc_decode(stream, 1, h, w, out=out)
                        except binding.PccError as e:
                            wrong.append(e)
                workers = [threading.Thread(target=work, args=a) for a in zip(cs, streams, outs)]
                start = time.perf_counter()
                for t in workers:
                    t.start()
                for t in workers:
                    t.join()
                seconds[variant] = time.perf_counter() - start
                torch.cuda.synchronize()
                assert not wrong and all(torch.equal(out, one) for out in outs)
            ratios.append(seconds["0"] / seconds["1"])
    finally:
        for c in sum(codecs.values(), []):
            c.close()
    print("%d threads, %dx%d: chosen against bands of 16 rows %s" % (threads, w, h, " ".join("%.3f" % r for r in ratios)), flush=True)
    if h * w > 1 << 20:                # (the small ones take a few ms: only their images are looked at)
        assert sorted(ratios)[2] <= 1.15


@pytest.mark.parametrize("net", ["paper", "diagonal"])
def test_a_decode_leaves_units_for_another(net):
    """Two threads decode four images of 768x512 each.  With the paper's network the one that starts alone takes bands of eight
    rows, 256 of them, of which 33 of an image's 64 can run at a time: with a workgroup for each of those the other one finds
    units.  (With one for every band it found none until the first bands had ended, after a third of the decode.)  In diagonal
    order all of them run at a time, so it takes bands of 16 rows."""
    from paper_2212_01185_amd import binding
    imgs = torch.from_numpy(np.random.default_rng(89).integers(0, 256, (4, 512, 768, 3), dtype=np.uint8)).cuda()
    codecs = [binding.Codec(BLOBS[net](0), 0) for _ in range(2)]
    outs = [torch.zeros_like(imgs) for _ in codecs]
    ratios = []
    try:
        stream = codecs[0].pcc_encode(imgs)
        for c, out in zip(codecs, outs):
            c.pcc_decode(stream, 4, 512, 768, out=out)
        for _ in range(7):
            streams = [torch.cuda.Stream() for _ in codecs]
            torch.cuda.synchronize()

            def work(c, s, out):
                with torch.cuda.stream(s):
                    c.pcc_decode(stream, 4, 512, 768, out=out)
            seconds = []
            for count in (1, 2):
                workers = [threading.Thread(target=work, args=a) for a in list(zip(codecs, streams, outs))[:count]]
                start = time.perf_counter()
                for t in workers:
                    t.start()
                for t in workers:
                    t.join()
                seconds.append(time.perf_counter() - start)
            ratios.append(seconds[1] / seconds[0])
            assert all(torch.equal(out, imgs) for out in outs)
    finally:
        for c in codecs:
            c.close()
    print("%s: two decodes against one %s" % (net, " ".join("%.3f" % r for r in ratios)), flush=True)
    assert sorted(ratios)[3] <= 1.25
