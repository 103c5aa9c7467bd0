"""fp16 pointwise kernels with large register tiles, at sizes on each side of the tile rules
and with partial pixel tiles: the folded patch embed + fuse and upsample + fuse (C = 128, 256,
384, 512), the two halves of a wide DC block in both forms, the strips of the wide depthwise, and
the reconstruction.  One frame through encoder and decoder, teacher-forced against the
oracle's float64 from the GPU's symbols, within the fp16 tolerance of the parity tests."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import codec_float as cf
from paper_2502_20762_amd.ncodec import Codec

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


def close(got, want, what):
    # the parity tests' bound for fp16 features and frames
    err = np.abs(got - want) / np.maximum(1.0, np.abs(want))
    assert err.max() <= 2e-2, (what, float(err.max()))


@pytest.mark.parametrize("H,W,C,block", [
    (16, 16, 128, "lrelu"),      # 4 pixels at 1/8, one at 1/16
    (80, 208, 128, "lrelu"),     # 260 pixels: partial tiles of 64 and 128
    (256, 400, 128, "lrelu"),
    (144, 144, 256, "lrelu"),
    (48, 80, 384, "gated"),
    (160, 272, 384, "lrelu"),    # 128-row passes (N = 384)
    (96, 176, 512, "lrelu"),
    (640, 704, 512, "lrelu"),    # 7,040 pixels: 128-pixel tiles, strips of 8 x 2
    (640, 704, 512, "gated"),
])
def test_frame_against_the_oracle(H, W, C, block):
    flat = synth.make_weights(C, 1, 1, block=block)
    p = oracle.unpack(flat, C, 1, 1, block=block)
    enc, dec = (Codec(H, W, C, 1, 1, "fp16", flat, device=DEV, block=block) for _ in range(2))
    rng = np.random.default_rng(H + W + C)
    feat = rng.standard_normal((C, H // 8, W // 8)).astype(np.float16)
    yhat = rng.standard_normal((C, H // 16, W // 16)).astype(np.float16)
    for c in (enc, dec):
        c.set_state(torch.from_numpy(feat).to(DEV), torch.from_numpy(yhat).to(DEV))
    x = synth.random_frame(H, W, seed=90)
    print("[gpu-pwt]", H, W, C, block, flush=True)
    q, _ = enc.encode(torch.from_numpy(x).to(DEV))
    st = cf.State(feat.astype(np.float64), yhat.astype(np.float64))
    y = cf.analysis(p, x, st.feat)
    mu, _ = cf.prior(p, st.yhat)
    # a symbol may differ from round(y - mu) only where y - mu is near a tie
    off = np.abs(host(q) - (y - mu))
    assert (off <= 0.5 + 2e-2 * np.maximum(1.0, np.abs(y))).all(), float(off.max())
    xr, after = cf.decode_frame(p, host(q), st)
    close(host(dec.decode(q)), xr, "frame")
    for c in (enc, dec):
        f, yh = (host(v) for v in c.get_state())
        close(f, after.feat, "f_t")
        close(yh, after.yhat, "yhat")
