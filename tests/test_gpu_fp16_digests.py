"""fp16 results stay what they were: an fp16 stream only decodes to what its encoder saw if both run the
same sums and roundings, also when one of them is an older build.  golden/fp16_digests.json
holds CRC-32s of one P-frame's symbols, rate and state and of a decoded frame, computed on an
MI355X with the kernels of commit d8d944d (one launch per block and chained alike), for every
width and block form, at sizes on both sides of the rules that choose tiles.  Bit for bit: no
tolerance.  Then infinities: a depthwise whose window holds one gives infinity, not NaN."""
import json
import os
import zlib

import numpy as np
import pytest
import torch

import synth
from paper_2502_20762_amd.ncodec import Codec

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
with open(os.path.join(os.path.dirname(__file__), "golden", "fp16_digests.json")) as f:
    DIGESTS = json.load(f)


def crc(t):
    return zlib.crc32(np.ascontiguousarray(t.cpu().numpy()).tobytes())


@pytest.mark.parametrize("d", DIGESTS, ids=lambda d: f"{d['height']}x{d['width']}-{d['channels']}-{d['block']}")
def test_results_are_bit_identical(d):
    H, W, C, ne, nd = d["height"], d["width"], d["channels"], d["enc"], d["dec"]
    flat = synth.make_weights(C, ne, nd, block=d["block"], n_fe=d["fe"], n_rg=d["rg"])
    rng = np.random.default_rng(H + W + C)
    feat = torch.from_numpy(rng.standard_normal((C, H // 8, W // 8)).astype(np.float16)).to(DEV)
    yhat = torch.from_numpy(rng.standard_normal((C, H // 16, W // 16)).astype(np.float16)).to(DEV)
    x = torch.from_numpy(synth.random_frame(H, W, seed=5)).to(DEV)
    q0 = torch.from_numpy(rng.integers(-3, 4, (C, H // 16, W // 16)).astype(np.int16)).to(DEV)
    for chains in (True, False):
        c = Codec(H, W, C, ne, nd, "fp16", flat, device=DEV, block=d["block"], n_fe_blocks=d["fe"], n_rg_blocks=d["rg"])
        c.block_chains(chains)
        c.set_state(feat, yhat)
        q, bits = c.encode(x)
        f, y = c.get_state()
        c.set_state(feat, yhat)
        frame = c.decode(q0)
        f2, _ = c.get_state()
        torch.cuda.synchronize()
        got = {"q": crc(q), "bits": float(bits).hex(), "feat": crc(f), "yhat": crc(y), "frame": crc(frame),
               "feat_decoded": crc(f2)}
        assert got == {k: d[k] for k in got}, "chains" if chains else "one launch per block"


@pytest.mark.parametrize("C", [64, 128])
def test_infinite_activations_stay_infinite(C):
    # every weight and bias positive; one infinite value in the context reaches the block through
    # the fuse conv, so the block's output is +inf in the 8 pixels around it and finite elsewhere (at
    # the pixel itself the residual is added through an identity matrix: 0 * inf)
    H, W = 80, 144
    flat = np.abs(synth.make_weights(C, 1, 1))
    flat = np.where(flat == 0, np.float32(2.0 ** -14), flat)
    feat = torch.zeros((C, H // 8, W // 8), dtype=torch.float16, device=DEV)
    feat[3, 4, 7] = float("inf")
    c = Codec(H, W, C, 1, 1, "fp16", flat, device=DEV)
    c.set_state(feat, torch.zeros((C, H // 16, W // 16), dtype=torch.float16, device=DEV))
    c.decode(torch.zeros((C, H // 16, W // 16), dtype=torch.int16, device=DEV))
    f, _ = c.get_state()
    torch.cuda.synchronize()
    want = torch.zeros((H // 8, W // 8), dtype=torch.bool)
    want[3:6, 6:9] = True
    f = f.cpu()
    assert not f[:, 4, 7].isfinite().any()
    want[4, 7] = False
    f[:, 4, 7] = 0
    assert not f.isnan().any()
    assert torch.equal(f == float("inf"), want.expand(C, -1, -1))
