"""The three containers of a two-step frame, encoded in one launch, against the oracle's coder
byte for byte: sections of one stream and of several with a ragged last one, the coder in line
and on the second stream.  Whole numbers: no tolerance."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import codec_int as ci
from oracle import entropy as E
from oracle import hyperprior as hp
from paper_2502_20762_amd.ncodec import Codec, _capacity

pytestmark = pytest.mark.gpu


# half of the latent: 256 symbols (z: 64), 1 stream; 3 full streams + 2,304; 5 + 4,096 (z: 2)
@pytest.mark.parametrize("H,W,C,par", [(32, 32, 128, False), (224, 480, 128, True), (352, 512, 128, False)])
def test_sections_match_oracle(H, W, C, par):
    flat = synth.make_weights(C, 1, 1, hyper=True)
    p = oracle.unpack(flat, C, 1, 1, hyper=True)
    ip, ih = ci.integerize(p), hp.integerize_hyper(p)
    enc = Codec(H, W, C, 1, 1, "int16", flat, device="cuda:0", hyperprior=True)
    enc.parallel_coding(par)
    x = synth.random_frame(H, W, seed=H)
    buf, nb = enc.encode_coded(torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0"))
    torch.cuda.synchronize()
    data, lens = buf.cpu().numpy(), nb.cpu().numpy()
    r = hp.encode_frame_int(p, ip, ih, x, ci.zero_state(ip, H, W))
    kz = np.broadcast_to(E.scale_index(hp.z_sigma(p))[:, None, None], r.sym.qz.shape)
    off = 0
    for i, (q, k) in enumerate([(r.sym.qz, kz), (r.sym.q1, E.scale_index(r.sigma1)),
                                (r.sym.q2, E.scale_index(r.sigma2))]):
        print("[gpu-sections]", (H, W), "container", i, "streams", -(-q.size // E.STREAM), flush=True)
        assert data[off:off + int(lens[i])].tobytes() == E.encode(q, k), f"container {i}"
        off += _capacity(q.size)
