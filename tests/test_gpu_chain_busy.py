"""Chains on a device that another stream keeps busy: a context codes the same frame again and again while
a second context's kernels (one launch per block, another form) come and go on its own stream; symbols
and state are bit for bit those of the context alone.  The edge pixels that tiles exchange are
stored from registers that the next instructions write, which shows only when other waves delay the store."""
import threading

import pytest
import torch

import synth
from paper_2502_20762_amd.ncodec import Codec, ncodec_get_state

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("path,H,W,C,block,n", [
    ("int16", 1088, 1920, 256, "gated", 4),
    ("int16", 544, 992, 256, "gated", 6),
    ("int16", 1088, 1920, 256, "lrelu", 3),
    ("int16", 480, 832, 128, "gated", 6),
    ("int16", 480, 832, 64, "lrelu", 6),
    ("fp16", 720, 1280, 256, "gated", 6),
    ("fp16", 1088, 1920, 256, "lrelu", 3),
    ("fp16", 480, 832, 128, "lrelu", 6),
    ("fp16", 480, 832, 64, "gated", 6),
])
def test_same_results_beside_another_stream(path, H, W, C, block, n):
    c = Codec(H, W, C, n, n, path, synth.make_weights(C, n, n, block=block), device=DEV, stream=torch.cuda.Stream(), block=block)
    other = Codec(1088, 1920, 256, 4, 4, "fp16", synth.make_weights(256, 4, 4), device=DEV, stream=torch.cuda.Stream())
    other.block_chains(False)
    x = torch.from_numpy(synth.random_frame(H, W, seed=1)).to(DEV)
    xo = torch.from_numpy(synth.random_frame(1088, 1920, seed=2)).to(DEV)
    print("[gpu-chain-busy]", path, H, W, C, block, flush=True)
    N = 30
    q, f = (torch.empty((N + 1, *s), dtype=dt, device=DEV) for s, dt in ((c.y_shape, torch.int16), (c.feat_shape, c.state_dtype)))
    y = torch.empty(c.y_shape, dtype=c.state_dtype, device=DEV)
    qo = torch.empty(other.y_shape, dtype=torch.int16, device=DEV)
    torch.cuda.synchronize()

    def code(k):
        c.reset()
        c.encode(x, q[k], want_bits=False)
        ncodec_get_state(c.ctx, f[k].data_ptr(), y.data_ptr())

    code(N)
    c.stream.synchronize()
    done = threading.Event()

    def busy():
        for k in range(3000):
            if done.is_set():
                break
            other.encode(xo, qo, want_bits=False)
            if k % 20 == 0:
                other.stream.synchronize()

    t = threading.Thread(target=busy)
    t.start()
    for k in range(N):
        code(k)
    c.stream.synchronize()
    done.set()
    t.join()
    torch.cuda.synchronize()
    assert c.block_chain_status() == (1, 0)
    bad = [k for k in range(N) if not (torch.equal(q[k], q[N]) and torch.equal(f[k], f[N]))]
    assert not bad, f"{len(bad)} of {N} frames differ"
