"""A chain launch without room for all of its tiles: forced (every launch is sealed by the first
workgroup that ends block 0), the blocks run one after the other by the workgroups that are there,
in every kernel form, with the encoder's downsample in the launch and with more tiles than
workgroups; symbols, rate, state and frames are bit for bit those of one launch per block, no wait
gives up, and chains that follow in the same context go on as before (direct and as graph replays)."""
import numpy as np
import pytest
import torch

import synth
from paper_2502_20762_amd.ncodec import Codec, load_library

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SEALED = 0x5EA1ED


def run(enc, dec, frames, mode):
    out = []
    for c in (enc, dec):
        assert load_library().ncodec_block_chains(c.ctx, mode) == 0
        c.reset()
    for x in frames:
        q, bits = enc.encode(x)
        xh = dec.decode(q)
        f, y = enc.get_state()
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (q, bits, xh, f, y)])
    for c in (enc, dec):
        assert c.block_chain_status()[1] == 0, "a wait gave up"
    return out


def same(a, b, what):
    for t, (u, v) in enumerate(zip(a, b)):
        for n, p, q in zip(("q", "bits", "xhat", "f_t", "yhat"), u, v):
            np.testing.assert_array_equal(p, q, err_msg=f"{what}, frame {t}: {n}")


@pytest.mark.parametrize("path,H,W,C,block,ne,nd", [
    ("fp16", 64, 64, 64, "lrelu", 4, 4),        # one tile
    ("int16", 112, 208, 64, "gated", 4, 5),
    ("fp16", 480, 832, 128, "lrelu", 6, 6),
    ("int16", 480, 832, 128, "lrelu", 6, 6),
    ("fp16", 112, 208, 128, "gated", 5, 4),
    ("fp16", 272, 400, 256, "gated", 2, 16),    # the downsample in the encoder's chain
    ("int16", 272, 400, 256, "gated", 4, 5),
    ("fp16", 1088, 1920, 256, "lrelu", 3, 2),   # 8 x 16 tiles
    ("int16", 1088, 1920, 256, "lrelu", 3, 2),  # 510 tiles
])
def test_sealed_launches_give_the_same(path, H, W, C, block, ne, nd):
    flat = synth.make_weights(C, ne, nd, block=block)
    enc, dec = (Codec(H, W, C, ne, nd, path, flat, device=DEV, block=block) for _ in range(2))
    frames = [torch.from_numpy(synth.random_frame(H, W, seed=s)).to(DEV) for s in (80, 81, 82)]
    print("[gpu-chain-seal]", path, H, W, C, block, flush=True)
    want = run(enc, dec, frames, 0)
    same(run(enc, dec, frames, SEALED), want, "sealed")
    assert enc.block_chain_status() == (1, 0)
    same(run(enc, dec, frames, 1), want, "chains after sealed ones")
    for c in (enc, dec):
        c.graphs(True)
    same(run(enc, dec, frames, SEALED), want, "sealed, replayed")
    same(run(enc, dec, frames, 1), want, "chains, replayed")
