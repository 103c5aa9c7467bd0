"""State layout conversion (ncodec_set_state / ncodec_get_state): planar to the context's
channels-last layout and back returns every value, at sizes with whole and partial
64-pixel tiles, rows that are and are not 16-byte aligned (pixel counts that are and are
not multiples of 8), every channel count, and buffers off 16-byte alignment."""
import pytest
import torch

import synth
from paper_2502_20762_amd.ncodec import Codec, ncodec_get_state, ncodec_set_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("H,W,C,path,shift", [
    (16, 16, 64, "int16", 0),     # 4 pixels at 1/8, one at 1/16
    (64, 64, 64, "fp16", 0),      # one whole tile; 16 pixels at 1/16
    (48, 80, 128, "int16", 0),    # 60 pixels: a partial tile, 15 at 1/16 (not a multiple of 8)
    (48, 80, 128, "fp16", 1),
    (272, 400, 256, "int16", 3),  # 1700 and 425 pixels, off alignment
    (64, 96, 512, "fp16", 0),
])
def test_state_round_trip(H, W, C, path, shift):
    c = Codec(H, W, C, 1, 1, path, synth.make_weights(C, 1, 1), device=DEV)
    g = torch.Generator(device=DEV).manual_seed(H + W + C)

    def planar(shape):
        n = shape[0] * shape[1] * shape[2]
        v = torch.randint(-30000, 30000, (n + shift,), generator=g, device=DEV, dtype=torch.int32).to(torch.int16)
        v = v[shift:].view(c.state_dtype)
        return v.reshape(shape)

    feat, yhat = planar(c.feat_shape), planar(c.y_shape)
    c.set_state(feat, yhat)
    for got, want in zip(c.get_state(), (feat, yhat)):
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))


def test_state_one_tensor_and_reset():
    c = Codec(112, 208, 64, 1, 1, "int16", synth.make_weights(64, 1, 1), device=DEV)
    g = torch.Generator(device=DEV).manual_seed(3)
    f, y = (torch.randint(-30000, 30000, s, generator=g, device=DEV, dtype=torch.int32).to(torch.int16)
            for s in (c.feat_shape, c.y_shape))
    c.set_state(f, y)
    # one tensor at a time (the other pointer NULL) leaves the other alone
    f2 = f.flip(0).contiguous()
    ncodec_set_state(c.ctx, f2.data_ptr(), 0)
    got = torch.zeros_like(y)
    ncodec_get_state(c.ctx, 0, got.data_ptr())
    assert torch.equal(got, y) and torch.equal(c.get_state()[0], f2)
    y2 = y.flip(0).contiguous()
    ncodec_set_state(c.ctx, 0, y2.data_ptr())
    assert torch.equal(c.get_state()[0], f2) and torch.equal(c.get_state()[1], y2)
    ncodec_set_state(c.ctx, 0, 0)
    assert torch.equal(c.get_state()[0], f2)
    c.reset()
    assert all(int(t.abs().max()) == 0 for t in c.get_state())
