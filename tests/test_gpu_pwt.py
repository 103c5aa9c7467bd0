"""fp16 pointwise kernels with large register tiles and the wide depthwise, at sizes on each side of the
rules that choose their tiles and with partial pixel tiles: the folded patch embed + fuse and upsample
+ fuse (C = 128, 256, 384, 512), the two halves of a wide DC block in both forms, the strips of
the wide depthwise (both paths), and the reconstruction.  variants() restates the rules, and a
test holds the list of sizes to every kernel that a rule can pick.  One frame through encoder and
decoder, teacher-forced against the oracle's float64 from the GPU's symbols, within the fp16
tolerance of the parity tests; the int path bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import codec_float as cf
from oracle import codec_int as ci
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


SIZES = [
    (16, 16, 64, "lrelu"),       # 4 pixels at 1/8, one at 1/16
    (16, 16, 128, "lrelu"),
    (80, 208, 128, "lrelu"),     # 260 pixels: partial tiles of 64 and 128
    (256, 400, 128, "lrelu"),
    (1072, 1488, 128, "lrelu"),  # 24,924 pixels: 134 x 186, cut by every tile and strip
    (144, 144, 256, "lrelu"),
    (528, 1200, 256, "lrelu"),   # 9,900
    (1072, 1488, 256, "lrelu"),
    (1616, 1968, 256, "lrelu"),  # 49,692
    (48, 80, 384, "gated"),
    (160, 272, 384, "lrelu"),    # 128-row passes (N = 384)
    (832, 992, 384, "lrelu"),    # 12,896
    (1072, 1488, 384, "lrelu"),
    (96, 176, 512, "lrelu"),
    (640, 704, 512, "lrelu"),    # 7,040
    (640, 704, 512, "gated"),
    (1200, 1776, 512, "lrelu"),  # 33,300: 150 x 222
    (1072, 1488, 512, "gated"),
]


def variants(H, W, C, block):
    """(layer, rows / 128, pixels / 32) of the pointwise kernels, ("dw", strip rows) of the wide depthwise."""
    p8 = (H // 8) * (W // 8)
    out = []

    def pick(layer, n, p):
        def wgs(rt, pg):
            return -(-p // (32 * pg)) * (n // (128 * rt))

        rows256 = n % 256 == 0 and (layer != "up" or C % 256 == 0)
        if layer == "gate":
            t = (2, 4) if wgs(2, 4) >= 384 else (2, 2)
        elif rows256 and wgs(2, 4) >= (512 if layer == "up" else 384):
            t = (2, 4)
        elif layer == "rec" and wgs(2, 2) >= 384:
            t = (2, 2)
        elif layer not in ("rec", "up") and wgs(1, 4) >= 384:
            t = (1, 4)
        else:
            t = (1, 2)
        out.append((layer, *t))

    pick("rec", 256, p8)
    if C % 128 == 0:
        pick("embed", C, p8)
        pick("up", 4 * C, p8 // 4)
    if C > 256:
        pick("gate" if block == "gated" else "lrelu", 2 * C, p8)
        pick("resid", C, p8)
        def dw(rows, cols):
            n = -(-(-(-(H // 8) // rows) * -(-(W // 8) // cols) * (C // 8)) // 256)
            return -(-n // 8) * 8

        out.append(("dw", 8 if dw(8, 2) >= 256 else 2 if dw(2, 1) > 384 else 1))
    return set(out)


def test_sizes_reach_every_variant():
    got = set().union(*(variants(*s) for s in SIZES))
    want = {(l, *t) for l, ts in {"rec": ((2, 4), (2, 2), (1, 2)), "embed": ((2, 4), (1, 4), (1, 2)), "up": ((2, 4), (1, 2)),
                                  "lrelu": ((2, 4), (1, 4), (1, 2)), "resid": ((2, 4), (1, 4), (1, 2)),
                                  "gate": ((2, 4), (2, 2))}.items() for t in ts} | {("dw", r) for r in (8, 2, 1)}
    assert got == want, (want - got, got - want)


S, MARGIN = 14, 2  # latent pixels of a crop, and of its border that a block's depthwise makes wrong


def crops(H, W):
    """Windows (in latent pixels) that the oracle is run on: the whole frame, or its corners and a window inside;
    slices of the window in latents, 1/8 grid and frame, and of the part inside it that no cut edge reaches."""
    h, w = H // 16, W // 16
    if h * w <= 500:
        at = [(0, 0, h, w)]
    else:
        at = [(y, x, S, S) for y, x in ((0, 0), (0, w - S), (h - S, 0), (h - S, w - S), (h // 3, w // 2 - 5))]
    for y, x, n, m in at:
        y0, x0 = MARGIN if y else 0, MARGIN if x else 0
        y1, x1 = n - (MARGIN if y + n < h else 0), m - (MARGIN if x + m < w else 0)
        yield [((slice(None), slice(f * y, f * (y + n)), slice(f * x, f * (x + m))),
                (slice(None), slice(f * y0, f * y1), slice(f * x0, f * x1))) for f in (1, 2, 16)]


@pytest.mark.parametrize("H,W,C,block", SIZES)
def test_frame_against_the_oracle(H, W, C, block):
    flat = synth.make_weights(C, 1, 1, block=block)
    p = oracle.unpack(flat, C, 1, 1, block=block)
    enc, dec = (Codec(H, W, C, 1, 1, "fp16", flat, device=DEV, block=block) for _ in range(2))
    rng = np.random.default_rng(H + W + C)
    feat = rng.standard_normal((C, H // 8, W // 8), dtype=np.float32).astype(np.float16)
    yhat = rng.standard_normal((C, H // 16, W // 16), dtype=np.float32).astype(np.float16)
    for c in (enc, dec):
        c.set_state(torch.from_numpy(feat).to(DEV), torch.from_numpy(yhat).to(DEV))
    x = synth.random_frame(H, W, seed=90)
    print("[gpu-pwt]", H, W, C, block, flush=True)
    q, _ = enc.encode(torch.from_numpy(x).to(DEV))
    q, frame = host(q), host(dec.decode(q))
    states = [[host(v) for v in c.get_state()] for c in (enc, dec)]
    for (l, li), (f, fi), (px, pxi) in crops(H, W):
        st = cf.State(feat[f].astype(np.float64), yhat[l].astype(np.float64))
        y = cf.analysis(p, x[px], st.feat)
        mu, _ = cf.prior(p, st.yhat)
        # a symbol may differ from round(y - mu) only where y - mu is near a tie
        off = np.abs(q[l] - (y - mu))[li]
        assert (off <= 0.5 + 2e-2 * np.maximum(1.0, np.abs(y[li]))).all(), float(off.max())
        xr, after = cf.decode_frame(p, q[l], st)
        close(frame[px][pxi], xr[pxi], "frame")
        for ft, yh in states:
            close(ft[f][fi], after.feat[fi], "f_t")
            close(yh[l], after.yhat, "yhat")


@pytest.mark.parametrize("rows,H,W,block", [
    (8, 1072, 1488, "lrelu"),  # strips of 8 x 2 on 134 x 186 pixels: cut at the bottom (134 = 16 * 8 + 6)
    (8, 1072, 1488, "gated"),
    (2, 368, 656, "lrelu"),    # of 2 x 1 on 46 x 82
    (1, 384, 512, "lrelu"),    # the largest launch of single pixels
    (1, 48, 80, "gated"),
])
def test_wide_depthwise_strips_int_bit_exact(rows, H, W, block):
    C = 512
    assert ("dw", rows) in variants(H, W, C, block)
    flat = synth.make_weights(C, 1, 1, block=block)
    p = oracle.unpack(flat, C, 1, 1, block=block)
    ip = ci.integerize(p)
    enc, dec = (Codec(H, W, C, 1, 1, "int16", flat, device=DEV, block=block) for _ in range(2))
    x = synth.random_frame(H, W, seed=91)
    print("[gpu-pwt] int16", H, W, C, block, flush=True)
    q, _ = enc.encode(torch.from_numpy(x).to(DEV))
    q, frame, ft = (host(v).astype(np.int64) for v in (q, dec.decode(q), dec.get_state()[0]))
    for (l, li), (f, fi), (px, pxi) in crops(H, W):
        h, w = l[1].stop - l[1].start, l[2].stop - l[2].start
        st = ci.zero_state(ip, 16 * h, 16 * w)
        r = ci.encode_frame(ip, x[px], st)
        np.testing.assert_array_equal(q[l][li], r.q[li])
        xr, after = ci.decode_frame(ip, q[l], st)
        np.testing.assert_array_equal(frame[px][pxi], xr[pxi])
        np.testing.assert_array_equal(ft[f][fi], after.feat[fi])
