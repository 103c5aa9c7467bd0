"""The workloads whose speed is looked after: frames coded through the public entry points.

Each case is one configuration of the codec and one thing that a program does with it:

  encode   one P-frame of one of several streams that share an encoder: the stream's state goes
           into the context, the frame is coded to symbols and its rate
  decode   an intra frame and the P-frames after it, from their symbols, by a decoder that was
           just reset (random access, or a joining receiver)
  stream   an encoder and its decoder coding an intra frame and the P-frames after it (the loop
           of a live link); the state that both sides end with comes back too
  coded    one P-frame to its entropy-coded container, and a frame from a container (the two ends of
           a link): the one just made on the int path, on the fp16 path one received from a peer

Inputs are synthetic: random-init weights at the scale a trained model has, and smooth frames with
small global motion and sensor noise.  Symbols and states that a case starts from come from a plain
torch evaluation of the model here (class ``Model``), so they depend on the seed alone.  That class
is also what ``exact`` runs, in 64 bits: float64 for the fp16 path, exact integers for the int path.
"""
import math

import numpy as np
import torch

from paper_2502_20762_amd.ncodec import Codec

DEV = "cuda:0"
CZ = 64       # channels of the hyper latent
NUM_QP = 64   # rate points of the vector banks


def _case(name, op, path, height, width, channels, enc, dec, frames=1, block="lrelu", fe=0, rg=0, banks=False,
          hyper=False):
    return {"name": name, "op": op, "path": path, "height": height, "width": width, "channels": channels,
            "enc": enc, "dec": dec, "frames": frames, "block": block, "fe": fe, "rg": rg, "banks": banks,
            "hyper": hyper}


def listed():
    return [
        # the smallest calls, a thumbnail or preview stream: launches and latency are all there is
        _case("tiny_fp16_decode", "decode", "fp16", 64, 64, 64, 2, 2, frames=4),
        _case("tiny_int16_stream", "stream", "int16", 64, 64, 64, 2, 2, frames=2),
        # a call at WVGA with the light model: fewer tiles than compute units
        _case("wvga_fp16_encode", "encode", "fp16", 480, 832, 128, 6, 6),
        _case("wvga_int16_stream", "stream", "int16", 480, 832, 128, 6, 6, frames=2),
        # the headline workload, 1080p (padded to 1088 rows) with the base model, each direction and path
        _case("hd1080_fp16_encode", "encode", "fp16", 1088, 1920, 256, 8, 8),
        _case("hd1080_fp16_decode", "decode", "fp16", 1088, 1920, 256, 8, 8, frames=2),
        _case("hd1080_int16_stream", "stream", "int16", 1088, 1920, 256, 8, 8, frames=2),
        # ... and with the entropy coder, as a link sends it
        _case("hd1080_fp16_coded", "coded", "fp16", 1088, 1920, 256, 8, 8),
        # every conditional-coding module and the two-step entropy model, at a ragged size (68 x 124
        # pixels at 1/8, neither a multiple of a tile), bit-exact path
        _case("hd544_int16_modules_coded", "coded", "int16", 544, 992, 256, 8, 8, block="gated", fe=2, rg=2,
              banks=True, hyper=True),
        # the gated block of the base model at 720p
        _case("hd720_fp16_gated_decode", "decode", "fp16", 720, 1280, 256, 8, 8, frames=2, block="gated"),
        # the largest frame, and the large model's width
        _case("uhd4k_fp16_encode", "encode", "fp16", 2176, 3840, 256, 8, 8),
        _case("hd1080_c512_fp16_decode", "decode", "fp16", 1088, 1920, 512, 8, 8, frames=2),
    ]


def draw(rng):
    """A case of the same ranges: 64x64 to 4K, every width, path, block form and operation, 1 to 16 blocks a side."""
    while True:
        c = {"op": rng.choice(["encode", "decode", "decode", "stream", "coded"]),
             "path": rng.choice(["fp16", "int16"]),
             "height": 16 * round(math.exp(rng.uniform(math.log(4), math.log(136)))),
             "width": 16 * round(math.exp(rng.uniform(math.log(4), math.log(240)))),
             "channels": rng.choice([64, 128, 256, 256, 256, 384, 512]),
             "enc": round(math.exp(rng.uniform(0, math.log(16)))), "dec": round(math.exp(rng.uniform(0, math.log(16)))),
             "frames": 1, "block": rng.choice(["lrelu", "lrelu", "gated"]),
             "fe": rng.choice([0, 0, 0, 1, 2]), "rg": rng.choice([0, 0, 0, 1, 2]), "banks": rng.random() < 0.25,
             "hyper": rng.random() < 0.25}
        if c["op"] in ("decode", "stream"):
            c["frames"] = rng.randint(1, 4)
        if c["path"] == "fp16" and c["op"] == "stream":
            c["op"] = "decode"  # see tolerance(): a stream of fp16 symbols is not comparable past its first frame
        if c["hyper"]:
            if c["path"] == "fp16" and c["op"] != "decode":
                continue  # see tolerance()
            c["channels"] = max(c["channels"], 128)
            c["height"], c["width"] = -(-c["height"] // 32) * 32, -(-c["width"] // 32) * 32
        if work(c)["flops"] * (2 if c["path"] == "int16" else 1) <= 1.0e12:
            return c


# ---------------------------------------------------------------- inputs
_weights = {}  # the last few models, as a program has its model at hand


def model_weights(c):
    """The flat parameter list in the order of include/ncodec.h, every value exact in fp16."""
    C, gated = c["channels"], c["block"] == "gated"
    key = (C, gated, c["enc"], c["dec"], c["fe"], c["rg"], c["banks"], c["hyper"])
    if key in _weights:
        return _weights[key]
    rng = np.random.default_rng(2025)
    out = []

    def conv(n, k, gain=1.0):
        out.append(rng.standard_normal(n * k, dtype=np.float32) * np.float32(gain / math.sqrt(k)))
        out.append(rng.uniform(-0.1, 0.1, n).astype(np.float32))

    def blocks(count):
        for _ in range(count):
            conv(C, 9)
            conv(2 * C, C)
            conv(C, C if gated else 2 * C, 0.125)  # a small residual step keeps the recursion over frames bounded

    def bank(n, slope, scale=1.0):
        qp = np.arange(NUM_QP)[:, None]
        out.append((scale * 2.0 ** (slope * qp / 32) * np.exp(rng.uniform(-0.1, 0.1, (NUM_QP, n)))).reshape(-1))

    conv(C, 192)
    conv(C, 2 * C)
    blocks(c["enc"])
    conv(C, 4 * C)
    conv(2 * C, C)
    conv(4 * C, C)
    conv(C, 2 * C)
    blocks(c["dec"])
    conv(192, C)
    blocks(c["fe"])
    blocks(c["rg"])
    if c["banks"]:
        for slope in (-1, 1, 0, 0):
            bank(C, slope)
    if c["hyper"]:
        conv(CZ, 4 * C)
        conv(8 * C, CZ)
        conv(C, C // 2)
        bank(CZ, -1, 2.0)
    flat = np.concatenate(out).astype(np.float16).astype(np.float32)
    while len(_weights) >= 16:
        _weights.pop(next(iter(_weights)))
    _weights[key] = flat
    return flat


def frames_of(c, seed, count):
    """`count` fp16 frames (3, H, W): sinusoids and noise, then small shifts of it with new noise."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    u = lambda a, b, *s: a + (b - a) * torch.rand(s, generator=g, device=DEV)  # noqa: E731
    H, W = c["height"], c["width"]
    y, x = torch.arange(H, device=DEV)[:, None] / H, torch.arange(W, device=DEV)[None, :] / W
    v = torch.full((3, H, W), 0.5, device=DEV)
    for k in range(3):
        amp, fx, fy, ph = u(0.02, 0.08, 8), u(-8, 8, 8), u(-8, 8, 8), u(0, 2 * math.pi, 8)
        for i in range(8):
            v[k] += amp[i] * torch.sin(2 * math.pi * (fx[i] * x + fy[i] * y) + ph[i])
    v = (v + 0.02 * torch.randn((3, H, W), generator=g, device=DEV)).clamp(0, 1)
    out = [v.half()]
    r = np.random.default_rng(seed)
    for _ in range(count - 1):
        v = torch.roll(v, tuple(int(t) for t in r.integers(-4, 5, 2)), (1, 2))
        v = (v + 0.01 * torch.randn((3, H, W), generator=g, device=DEV)).clamp(0, 1)
        out.append(v.half())
    return out


# ---------------------------------------------------------------- the model in plain torch
class Model:
    """The transform of include/ncodec.h on (channels, pixels) tensors; int path in exact integers (as float64)."""

    def __init__(self, c, dtype):
        self.c, self.C, self.int = c, c["channels"], c["path"] == "int16"
        self.h, self.w = c["height"] // 8, c["width"] // 8
        self.dt = torch.float64 if self.int else dtype
        flat, at, C = torch.from_numpy(model_weights(c)).to(DEV, torch.float64), 0, self.C
        gated = c["block"] == "gated"

        def take(*shape):
            nonlocal at
            n = math.prod(shape)
            at += n
            return flat[at - n:at].reshape(shape)

        def conv(n, k):
            return [take(n, k), take(n)]

        def blocks(count):
            return [[conv(C, 9), conv(2 * C, C), conv(C, C if gated else 2 * C)] for _ in range(count)]

        self.pe, self.fuse_enc, self.enc = conv(C, 192), conv(C, 2 * C), blocks(c["enc"])
        self.down, self.head, self.up = conv(C, 4 * C), conv(2 * C, C), conv(4 * C, C)
        self.fuse_dec, self.dec, self.rec = conv(C, 2 * C), blocks(c["dec"]), conv(192, C)
        self.fe, self.rg = blocks(c["fe"]), blocks(c["rg"])
        if c["banks"]:  # a context starts at rate point 0, folded into the layers around
            qe, qd, qf, qr = [take(NUM_QP, C)[0] for _ in range(4)]
            f16 = lambda t: t.half().double()  # noqa: E731
            self.down = [f16(self.down[0] * qe[:, None]), f16(self.down[1] * qe)]
            self.up[0] = f16(self.up[0] * qd)
            self.rec[0] = f16(self.rec[0] * qr)
            for l in (self.fuse_enc, self.fuse_dec):
                l[0] = torch.cat([l[0][:, :C], f16(l[0][:, C:] * qf)], 1)
        if c["hyper"]:
            self.zana, self.zsyn, self.step2 = conv(CZ, 4 * C), conv(8 * C, CZ), conv(C, C // 2)
            self.zscale = take(NUM_QP, CZ)[0].clamp(min=0.11)
        every = [self.pe, self.fuse_enc, self.down, self.head, self.up, self.fuse_dec, self.rec]
        every += [l for b in self.enc + self.dec + self.fe + self.rg for l in b]
        every += [self.zana, self.zsyn, self.step2] if c["hyper"] else []
        for l in every:
            for i in (0, 1):
                l[i] = torch.round(l[i] * 8192).clamp(-32768, 32767) if self.int else l[i].to(self.dt)
        if self.int and gated:
            v = torch.arange(-32768, 32768, device=DEV, dtype=torch.float64)
            self.sig = torch.round(512 * torch.sigmoid(4 * v / 512))

    def sat(self, v):
        return v.clamp(-32768, 32767) if self.int else v

    def rescale(self, acc):
        return torch.round(acc / 8192).clamp(-32768, 32767) if self.int else acc

    def pw(self, l, x):
        return self.rescale(l[0] @ x + (512 * l[1] if self.int else l[1])[:, None])

    def dw(self, l, x):
        C, k = x.shape[0], l[0]
        p = torch.nn.functional.pad(x.reshape(C, self.h, self.w), (1, 1, 1, 1))
        acc = (512 * l[1] if self.int else l[1])[:, None, None] + torch.zeros((C, self.h, self.w), device=DEV, dtype=self.dt)
        for i in range(3):
            for j in range(3):
                acc += k[:, 3 * i + j, None, None] * p[:, i:i + self.h, j:j + self.w]
        return self.rescale(acc).reshape(C, -1)

    def blocks(self, bs, z):
        for dw, pw1, pw2 in bs:
            h = self.pw(pw1, self.dw(dw, z))
            if self.c["block"] == "gated":
                a, b = h[:self.C], h[self.C:]
                if self.int:
                    g = self.sat(torch.round(torch.round(a * self.sig[(a + 32768).long()] / 512) * b / 512))
                else:
                    g = a * torch.sigmoid(4 * a) * b
            else:
                g = torch.maximum(h, torch.round(819 * h / 8192) if self.int else 0.1 * h)
            z = self.sat(z + self.pw(pw2, g))
        return z

    def down2(self, l, x, h, w):
        """2x2 stride-2 conv of an h x w map."""
        C = x.shape[0]
        u = x.reshape(C, h // 2, 2, w // 2, 2).permute(0, 2, 4, 1, 3).reshape(4 * C, -1)
        return self.pw(l, u)

    def up2(self, l, x, h, w):
        """1x1 conv and pixel shuffle x2 of an h x w map."""
        v = self.pw(l, x)
        return v.reshape(-1, 2, 2, h, w).permute(0, 3, 1, 4, 2).reshape(v.shape[0] // 4, -1)

    def zero_state(self):
        z = lambda n: torch.zeros((self.C, n), device=DEV, dtype=self.dt)  # noqa: E731
        return z(self.h * self.w), z(self.h * self.w // 4)

    def rate(self, q, sigma):
        r, a = math.sqrt(0.5), q.double().abs()
        L = 0.5 * (torch.special.erfc((a - 0.5) * r / sigma) - torch.special.erfc((a + 0.5) * r / sigma))
        return -torch.log2(L.clamp(min=1e-9)).sum()

    def quantise(self, v, mu):
        return torch.round((v - mu) / 512) if self.int else torch.round(v - mu)

    def dequantise(self, q, mu):
        return self.sat(512 * q + mu) if self.int else q + mu

    def entropy(self, state, y=None, q=None):
        """Symbols (flat, z after y), their rate and yhat, from the latent y or from the symbols q."""
        C, n = self.C, self.h * self.w // 4
        ms = self.pw(self.head, state[1])
        bits, qz = 0.0, None
        if self.c["hyper"]:
            if y is not None:
                z = self.down2(self.zana, y, self.h // 2, self.w // 2)
                qz = self.quantise(z, 0.0)
            else:
                qz = q[C * n:].reshape(CZ, -1).to(self.dt)
            bits = bits + self.rate(qz, self.zscale[:, None])
            zhat = self.sat(512 * qz) if self.int else qz
            ms = self.sat(ms + self.up2(self.zsyn, zhat, self.h // 4, self.w // 4))
        mu, s = ms[:C], ms[C:]
        out, yhat = [], []
        halves = [(0, C // 2), (C // 2, C)] if self.c["hyper"] else [(0, C)]
        for k, (a, b) in enumerate(halves):
            m, t = mu[a:b], s[a:b]
            if k == 1:
                d = self.pw(self.step2, yhat[0])
                m, t = self.sat(m + d[:C // 2]), self.sat(t + d[C // 2:])
            qk = self.quantise(y[a:b], m) if y is not None else q[a * n:b * n].reshape(b - a, n).to(self.dt)
            t = t.double() / (512 if self.int else 1)
            bits = bits + self.rate(qk, torch.nn.functional.softplus(t, threshold=40).clamp(min=0.11))
            out.append(qk)
            yhat.append(self.dequantise(qk, m))
        q = torch.cat([v.reshape(-1) for v in out + ([qz] if qz is not None else [])]).to(torch.int16)
        return q, bits, torch.cat(yhat)

    def decoder(self, yhat, ctx):
        d = self.up2(self.up, yhat, self.h // 2, self.w // 2)
        return self.blocks(self.dec, self.pw(self.fuse_dec, torch.cat([d, ctx])))

    def encode(self, frame, state):
        """(symbols, bits, new state)"""
        ctx = self.blocks(self.fe, state[0])
        u = frame.to(self.dt).reshape(3, self.h, 8, self.w, 8).permute(0, 2, 4, 1, 3).reshape(192, -1)
        e = self.pw(self.pe, torch.round(512 * u) if self.int else u)
        z = self.blocks(self.enc, self.pw(self.fuse_enc, torch.cat([e, ctx])))
        q, bits, yhat = self.entropy(state, y=self.down2(self.down, z, self.h, self.w))
        return q, bits, (self.decoder(yhat, ctx), yhat)

    def decode(self, q, state):
        """(frame, new state)"""
        ctx = self.blocks(self.fe, state[0])
        _, _, yhat = self.entropy(state, q=q)
        f = self.decoder(yhat, ctx)
        v = self.pw(self.rec, self.blocks(self.rg, f)).clamp(0, 512 if self.int else 1)
        v = v.reshape(3, 8, 8, self.h, self.w).permute(0, 3, 1, 4, 2).reshape(3, 8 * self.h, 8 * self.w)
        return v, (f, yhat)

    def planar(self, state):
        """The state as the entry points take it."""
        dt = torch.int16 if self.int else torch.float16
        return (state[0].to(dt).reshape(self.C, self.h, self.w), state[1].to(dt).reshape(self.C, self.h // 2, self.w // 2))

    def flat(self, planar):
        return tuple(t.to(self.dt).reshape(self.C, -1) for t in planar)


def start_of(c, seed):
    """What a case begins with: frames, and the symbols (decode) or the state after the intra frame (encode, coded)."""
    if c["op"] == "stream":
        return {"frames": frames_of(c, seed, c["frames"])}
    m = Model(c, torch.float32)
    frames = frames_of(c, seed, c["frames"] if c["op"] == "decode" else 2)
    state, symbols = m.zero_state(), []
    for x in frames if c["op"] == "decode" else frames[:1]:
        q, _, state = m.encode(x, state)
        symbols.append(q)
    return {"frames": frames, "symbols": symbols, "state": m.planar(state)}


def prepare(case, seed):
    s = start_of(case, seed)
    c, w = case, model_weights(case)

    def codec():
        return Codec(c["height"], c["width"], c["channels"], c["enc"], c["dec"], c["path"], w, device=DEV,
                     block=c["block"], n_fe_blocks=c["fe"], n_rg_blocks=c["rg"], qp_banks=c["banks"],
                     hyperprior=c["hyper"])

    s["case"], op = c, c["op"]
    if op != "decode":
        s["enc"] = codec()
    if op != "encode":
        s["dec"] = codec()
    any_ = s.get("enc") or s["dec"]
    e = lambda shape, dt: torch.empty(shape, dtype=dt, device=DEV)  # noqa: E731
    n = c["frames"]
    s["q"] = [e(any_.q_shape, torch.int16) for _ in range(n)]
    s["bits"] = [e((), torch.float64) for _ in range(n)]
    if op == "decode":
        s["symbols"] = [q.reshape(any_.q_shape).contiguous() for q in s["symbols"]]
    if op != "encode":
        s["out"] = [e(any_.frame_shape, any_.state_dtype) for _ in range(n)]
    if op == "coded":
        s["stream"] = torch.zeros((any_.stream_capacity(),), dtype=torch.uint8, device=DEV)
        if c["path"] == "fp16":  # the peer's container, of the reference symbols of the same frame
            m = Model(c, torch.float32)
            q = m.encode(s["frames"][1], m.flat(s["state"]))[0].reshape(any_.q_shape)
            s["dec"].set_state(*s["state"])
            got, size = s["dec"].rans_encode(q, s["dec"].scale_indices())
            s["received"] = got, int(size)
    return s


def run(s):
    op, enc, dec = s["case"]["op"], s.get("enc"), s.get("dec")
    if op == "encode":
        enc.set_state(*s["state"])
        q, bits = enc.encode(s["frames"][1], s["q"][0], s["bits"][0])
        return {"q": q, "bits": bits}
    if op == "decode":
        dec.reset()
        return {"frames": [dec.decode(q, out) for q, out in zip(s["symbols"], s["out"])]}
    if op == "stream":
        enc.reset()
        dec.reset()
        for x, q, bits, out in zip(s["frames"], s["q"], s["bits"], s["out"]):
            enc.encode(x, q, bits)
            dec.decode(q, out)
        return {"q": s["q"], "bits": s["bits"], "frames": s["out"], "enc_state": enc.get_state(),
                "dec_state": dec.get_state()}
    enc.set_state(*s["state"])
    dec.set_state(*s["state"])
    stream, sizes = enc.encode_coded(s["frames"][1], s["stream"], q_out=s["q"][0], bits_out=s["bits"][0])
    sizes = sizes.reshape(-1).tolist()  # a program waits for them: they are what it sends
    two_step = s["case"]["hyper"]
    received = s.get("received") or (stream, stream.numel() if two_step else sizes[0])
    frame, status = dec.decode_coded(*received, s["out"][0])
    r = {"q": s["q"][0], "bits": s["bits"][0], "sizes": [float(n) for n in sizes], "frame": frame, "status": status}
    if s["case"]["path"] == "int16":
        r["containers"] = stream  # the containers at their fixed places, zeros from preparation behind each
    return r


def exact(case, seed):
    c = case
    s, m = start_of(c, seed), Model(c, torch.float64)
    # bits of the fp16 path: one number, a sum in which the roundings of the symbols cancel by chance, so its
    # distance from 64 bits says nothing on precision (tolerance() still holds it); the int path's is exact
    told = (lambda b: b) if m.int else (lambda b: None)
    if c["op"] == "encode":
        q, bits, _ = m.encode(s["frames"][1], m.flat(s["state"]))
        return {"q": q, "bits": told(bits)}
    if c["op"] == "decode":
        state, out = m.zero_state(), []
        for q in s["symbols"]:
            x, state = m.decode(q, state)
            out.append(x)
        return {"frames": out}
    if c["op"] == "stream":
        state, r = m.zero_state(), {"q": [], "bits": [], "frames": []}
        for x in s["frames"]:
            q, bits, after = m.encode(x, state)
            r["frames"].append(m.decode(q, state)[0])
            r["q"].append(q)
            r["bits"].append(told(bits))
            state = after
        r["enc_state"] = r["dec_state"] = m.planar(state)
        return r
    state = m.flat(s["state"])
    q, bits, _ = m.encode(s["frames"][1], state)
    if not m.int:  # the peer's symbols
        p = Model(c, torch.float32)
        q = p.encode(s["frames"][1], p.flat(s["state"]))[0]
    return {"q": q, "bits": told(bits), "frame": m.decode(q, state)[0]}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Multiply-adds of the layers (2 flops each); frames, symbols, containers, states and weights once each."""
    c, C = case, case["channels"]
    p8 = c["height"] * c["width"] // 64
    p16 = p8 // 4
    hid = C if c["block"] == "gated" else 2 * C
    block = p8 * (9 * C + 2 * C * C + hid * C)
    prior = p16 * 2 * C * C + (p16 // 4 * (4 * C * CZ + 8 * C * CZ) + p16 * C * C // 2 if c["hyper"] else 0)
    decoder = p16 * 4 * C * C + p8 * 2 * C * C + c["dec"] * block
    enc = p8 * (192 * C + 2 * C * C) + (c["fe"] + c["enc"]) * block + p16 * 4 * C * C + prior + decoder
    dec = prior + decoder + (c["fe"] + c["rg"]) * block + p8 * 192 * C
    frame, symbols, state = 3 * 64 * p8 * 2, p16 * C * 2 + (p16 // 4 * CZ * 2 if c["hyper"] else 0), (p8 + p16) * C * 2
    weights = 2 * (C * (192 + 2 * C) + 4 * C * C + 2 * C * C + 4 * C * C + 2 * C * C + 192 * C
                   + (c["enc"] + c["dec"] + c["fe"] + c["rg"]) * C * (9 + 2 * C + hid))
    n, op = c["frames"], c["op"]
    if op == "encode":
        return {"bytes": frame + symbols + 3 * state + weights, "flops": 2 * enc}
    if op == "decode":
        return {"bytes": n * (symbols + frame) + 2 * state + weights, "flops": 2 * n * dec}
    if op == "stream":
        return {"bytes": n * 2 * (frame + symbols) + 6 * state + 2 * weights, "flops": 2 * n * (enc + dec)}
    return {"bytes": 2 * (frame + symbols) + 6 * state + 2 * weights, "flops": 2 * (enc + dec)}


def tolerance(case):
    """int16: bit for bit, but for the rate, a sum of fp32 terms (3e-8 from 64 bits).  fp16: roundings of activations
    and weights to fp16 (2^-11 each) through all layers; over sizes, widths and depths frames are up to 8e-4 from the
    model in 64 bits (single pixels 6e-3 of the rms), rates 1e-4, and up to 5e-4 of the symbols, whose value lies that
    close to a tie, go the other way.  A flipped symbol moves the frames decoded from it by 2e-2 and, with the hyper
    latent, the distribution of the symbols around it, so fp16 symbols are compared for one frame from a given state,
    never decoded from, and without the hyper latent.  Each bound is about four times what was seen (and four
    symbols of the smallest frames)."""
    if case["path"] == "int16":
        return {"rel": 2e-7, "max": 2e-7, "differ": 0.0}
    symbols = case["height"] * case["width"] * case["channels"] // 256
    return {"rel": 3e-3, "max": 2.5e-2, "differ": max(2e-3, 4.0 / symbols)}
