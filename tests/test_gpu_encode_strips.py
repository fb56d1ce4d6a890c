"""The pixel kernel's strips of 32 pixels: sizes where a strip's bytes are gathered in another way (whole strips inside the image,
strips that touch its borders, ragged first strips, fewer pixels than a strip), for every network.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import pcc_oracle as po
from paper_2212_01185_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BLOBS = {"workload": synth.make_blob, "paper": synth.make_paper_blob, "diagonal": synth.make_diagonal_blob}
BLOBS.update({name: lambda seed, shape=shape: synth.make_ablation_blob(*shape, seed=seed) for name, shape in synth.ABLATION_SHAPES.items()})
# A strip lies inside when its first column is at least 2 and three more columns follow its last one: with strips dealt out from the
# right edge the first inside one appears at a width of 32 + 32 + 2 columns; heights 1 to 3 have no, no and one such row.
SIZES = [(3, 1), (1, 31), (3, 32), (2, 33), (4, 65), (3, 66), (4, 67), (5, 99), (3, 130)]


@pytest.mark.parametrize("net", sorted(BLOBS))
def test_head_outputs_and_bits_at_strip_borders(net):
    """All head outputs within 2e-3 of the exact network (the path's bound), bits/pixel within 0.1 %, the round trip exact."""
    from paper_2212_01185_amd import binding
    blob = BLOBS[net](0)
    codec, orc = binding.Codec(blob, 0), po.Oracle(blob)
    rng = np.random.default_rng(7)
    try:
        for n, (h, w) in enumerate(SIZES):
            imgs = rng.integers(0, 256, (1 + n % 3, h, w, 3), dtype=np.uint8)
            print("%s %dx%dx%d" % (net, len(imgs), h, w), flush=True)
            d = torch.from_numpy(imgs).cuda()
            params, bits = codec.pcc_encode_probs(d)
            stream = codec.pcc_encode(d)
            assert torch.equal(codec.pcc_decode(stream, len(imgs), h, w), d)
            got = params.cpu().numpy().astype(np.float64)
            for i, img in enumerate(imgs):
                assert np.abs(got[i] - orc.params_rows(img, range(h), po.MODE_EXACT)).max() <= 2e-3
            want = orc.encode(imgs, po.MODE_EXACT)[1]
            assert abs(float(bits.double().sum().item()) / want.sum() - 1) <= 1e-3
    finally:
        codec.close()
