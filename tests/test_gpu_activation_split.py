"""The decoder splits activations by two forms, on the matrix core and by the vector ALU, which differ from network to
network and from launch to launch, the encoder by a third, in pieces between its MFMAs: all must give the same bits, or a
stream could not be decoded.  Needs an MI355X."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2212_01185_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "device_checks", "libact_split_check.so")
FORMS = 6                                     # of act_split_check: matrix core, vector ALU, the encoder's four schedules
LARGEST_BF16 = np.uint32(0x7F7F7FFF)          # the largest float whose nearest bf16 is finite


def _log(msg):
    print(msg, flush=True)


def _bf16(x):
    """Bits of the nearest bf16 (ties to even) of finite floats."""
    bits = x.view(np.uint32).astype(np.uint64)
    return ((bits + 0x7FFF + ((bits >> 16) & 1)) >> 16).astype(np.uint32)


def _values():
    """Groups of four: activations of ordinary size, every exponent of either sign, values on and beside bf16's ties."""
    rng = np.random.default_rng(90)
    ordinary = rng.normal(0.0, 1.0, 1 << 21).astype(np.float32)
    any_bits = rng.integers(0, 1 << 32, 1 << 21, dtype=np.uint64).astype(np.uint32)
    ties = (rng.integers(0, 1 << 16, 1 << 18).astype(np.uint32) << 16) | rng.choice(
        np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], dtype=np.uint32), 1 << 18)
    special = np.array([0, 0x80000000, 1, 0x80000001, 0x00800000, LARGEST_BF16, LARGEST_BF16 | 0x80000000], dtype=np.uint32)
    bits = np.concatenate([any_bits, ties, np.resize(special, 1 << 10)])
    bits = np.where((bits & 0x7FFFFFFF) <= LARGEST_BF16, bits, bits & 0x80FFFFFF)
    return np.concatenate([ordinary, bits.view(np.float32)]).reshape(-1, 4)


@pytest.mark.parametrize("leaky", [False, True])
def test_both_forms_of_the_split_give_the_same_bits(leaky):
    """The decoder's two forms, and the encoder's pieces in each of their four schedules."""
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build_device_checks()
    lib = C.CDLL(LIB)
    lib.act_split_check.argtypes = [C.c_void_p, C.c_size_t, C.c_int, C.c_void_p, C.c_void_p]
    v = _values()
    d = torch.from_numpy(v).cuda()
    out = torch.zeros((len(v), FORMS * 4), dtype=torch.int32, device="cuda")
    rc = lib.act_split_check(d.data_ptr(), len(v), int(leaky), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = out.cpu().numpy().view(np.uint32).reshape(-1, FORMS, 4)
    for form in range(1, FORMS):
        np.testing.assert_array_equal(got[:, 0], got[:, form], err_msg="form %d" % form)
    # and they are what the split is defined as: hi the nearest bf16 of the activation, lo of what hi leaves
    act = np.where(v > 0, v, (np.float32(0.01) * v if leaky else np.float32(0))).astype(np.float32)
    hi = _bf16(act)
    lo = _bf16(act - (hi << 16).astype(np.uint32).view(np.float32))
    want = np.concatenate([hi[:, 0::2] | hi[:, 1::2] << 16, lo[:, 0::2] | lo[:, 1::2] << 16], axis=1)
    zero = np.uint32(0x7FFF7FFF)           # a zero's sign is nobody's: masked where a half is zero
    same = (got[:, 0] ^ want)
    for half in (0xFFFF, 0xFFFF0000):
        h = np.uint32(half)
        differ = ((same & h) != 0) & (((got[:, 0] | want) & h & zero) != 0)
        assert not differ.any(), (v[differ.any(axis=1)][:4], got[differ.any(axis=1)][:4], want[differ.any(axis=1)][:4])


def _overflowing(dims, layer):
    """He-initialised layers with hidden layer `layer` scaled up so far that some of its activations pass bf16's range and
    the next ones down again, and the layers that give the same numbers for a pixel that stays in range: all factors are
    powers of two.  (Behind the last hidden layer there is only the head, whose weights can be scaled down by 2^-100 without
    becoming subnormal: the head outputs are larger by the rest.)"""
    layers = [[w.copy(), b] for w, b in synth.make_weights(0, dims)]
    plain = [[w.copy(), b] for w, b in layers]
    up = 127
    layers[layer][0] *= np.float32(2.0 ** up)
    if layer + 2 < len(layers):
        layers[layer + 1][0] *= np.float32(2.0 ** -64)
        layers[layer + 2][0] *= np.float32(2.0 ** (64 - up))
    else:
        layers[layer + 1][0] *= np.float32(2.0 ** -100)
        plain[layer + 1][0] *= np.float32(2.0 ** (up - 100))
    return layers, plain


# network: layer widths, header, launches of its decoder (one and two workgroups per unit; 3: bands of eight rows)
NETS = {"workload": (synth.DEFAULT_DIMS, {}, "123"),
        "paper": (synth.PAPER_DIMS, dict(k=3, nbhd=12, delay=3, act=synth.ACT_LEAKY), "123"),
        "more_filters": (synth.ablation_dims(3, 192, 5), dict(k=3, nbhd=12, delay=3, act=synth.ACT_LEAKY), "123"),
        "more_mixtures": (synth.ablation_dims(5, 128, 5), dict(k=5, nbhd=12, delay=3, act=synth.ACT_LEAKY), "3"),
        "most_mixtures": (synth.ablation_dims(7, 128, 5), dict(k=7, nbhd=12, delay=3, act=synth.ACT_LEAKY), "3")}


@pytest.mark.parametrize("net", sorted(NETS))
def test_roundtrip_where_activations_pass_the_range_of_bf16(net, monkeypatch):
    """An activation that rounds to infinity has different lo parts in the forms (the matrix core multiplies it with zero
    for its three neighbours), and the pixel is NaN from the next layer on: the same NaN in both, whose products are all
    0xFFC00000.  All decoders must return the image."""
    from paper_2212_01185_amd import binding
    dims, header, launches = NETS[net]
    rng = np.random.default_rng(91)
    imgs = torch.from_numpy(rng.integers(0, 256, (2, 37, 50, 3), dtype=np.uint8)).cuda()
    for layer in range(len(dims) - 2):
        layers, plain = (synth.pack_blob(x, **header) for x in _overflowing(dims, layer))
        c = binding.Codec(plain, 0)
        want = c.pcc_encode_probs(imgs)[0]
        c.close()
        for launch in launches:
            monkeypatch.setenv("PCC_DECODE_VARIANT", launch)
            c = binding.Codec(layers, 0)
            try:
                got = c.pcc_encode_probs(imgs)[0]
                share = (~(got == want).all(dim=-1)).float().mean().item()
                _log("%s, layer %d, launch %s: %.3f of the pixels out of range" % (net, layer, launch, share))
                assert 0.01 < share < 0.99
                stream = c.pcc_encode(imgs)
                assert torch.equal(c.pcc_decode(stream, 2, 37, 50), imgs)
            finally:
                c.close()
