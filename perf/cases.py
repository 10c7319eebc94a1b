"""Timed cases of the generator, through its public entry points.

Three kinds of pass: generation of audio (``WaveNet.generate``), teacher forcing of recorded audio
(``WaveNet.teacher_force``) and the conditioning network (``Conditioner`` and its
``condition_static``).  ``listed`` holds the sizes that a program meets in practice, ``draw`` picks
others of the same ranges, ``prepare`` makes what a program holds before a call (model handle,
inputs, output and state buffers), ``run`` is one pass, ``work`` the bytes and operations a pass
cannot do without, and ``exact`` the same outputs in 64 bits from plain torch.

A generation pass starts every stream from silence, generates T samples (in ``chunk``-step calls
that continue the state, as a streaming server makes them) and then forces one step, the splice into
recorded audio; that step's logits depend on every layer's history, so they show the whole state
beside the samples.
"""
import math

import numpy as np
import torch

import paper_1702_07825_amd as wn

A = 256                       # mu-law classes
SHAPES = ((16, 32), (32, 128), (64, 128), (64, 256), (128, 256))  # (r, s) pairs the library takes
DTYPES = ("f32", "bf16", "i8")
FEATURES, H1, FRAME_HZ = 227, 256, 256  # the paper's features per frame and the first QRNN layer's width
DEV = "cuda"


def _net(name, kind, l, r, s, B, T, dtype="f32", taps=1, cycle=10, chunk=0, rule="direct"):
    return {"name": name, "kind": kind, "l": l, "r": r, "s": s, "B": B, "T": T, "dtype": dtype, "taps": taps,
            "cycle": cycle, "chunk": chunk, "rule": rule}


def _cond(name, l, r, B, frames, audio_hz, static):
    return {"name": name, "kind": "cond", "l": l, "r": r, "B": B, "frames": frames, "audio_hz": audio_hz,
            "static": static}


def listed():
    return [
        # a device-sized voice: the smallest model, 0.1 s in one call
        _net("gen_l4_r16_b1", "gen", 4, 16, 32, 1, 1600, cycle=4),
        # live speech from one voice: 20 ms calls that continue each other
        _net("gen_l20_r64_b1_20ms", "gen", 20, 64, 256, 1, 1280, chunk=320),
        # one utterance offline (a quarter of a second of it): the headline model
        _net("gen_l20_r64_b1", "gen", 20, 64, 256, 1, 4000),
        # the deepest model of the paper, two-tap input convolution
        _net("gen_l40_r64_b1", "gen", 40, 64, 256, 1, 2000, taps=2),
        # a batch of utterances on the widest model
        _net("gen_l20_r128_b32", "gen", 20, 128, 256, 32, 800),
        # a server's full batch, bf16 weights
        _net("gen_l20_r64_b256_bf16", "gen", 20, 64, 256, 256, 160, dtype="bf16"),
        # an odd batch of an int8 model, softened sampling
        _net("gen_l20_r64_b37_i8", "gen", 20, 64, 256, 37, 333, dtype="i8", rule="temperature"),
        # scoring one second of recorded speech
        _net("tf_l20_r64_b1", "tf", 20, 64, 256, 1, 16000),
        # scoring a batch of short clips with the widest model
        _net("tf_l20_r128_b7", "tf", 20, 128, 256, 7, 1501),
        # a server warming 48 streams up on their prompts, bf16 weights
        _net("tf_l20_r64_b48_bf16", "tf", 20, 64, 256, 48, 2047, dtype="bf16"),
        # conditioning of one second of speech for the headline model, without a workspace
        _cond("cond_l20_r64_b1", 20, 64, 1, 256, 16000, True),
        # conditioning of a server's batch of two-second utterances
        _cond("cond_l20_r64_b32", 20, 64, 32, 512, 16000, False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("gen", "gen", "tf", "tf", "cond"))
    l = _log_int(rng, 4, 40)
    if kind == "cond":
        r = rng.choice((16, 32, 64, 128))
        frames, audio = _log_int(rng, 37, 700), rng.choice((16000, 16384, 48000))
        # at most the output of the largest listed case, and h2 = l r within the library's limit
        l = min(l, 8192 // r)
        steps = frames * audio // FRAME_HZ
        most = max(1, int(32 * 32000 * 20 * 128 // (steps * l * 2 * r)))
        B = _log_int(rng, 1, min(48, most))
        c = _cond("", l, r, B, frames, audio, False)
        c["static"] = B * frames * (6 * max(H1, l * r) + 2 * H1 + 2 * l * r) * 4 + 1024 <= wn.COND_SCRATCH_BYTES
    else:
        r, s = rng.choice(SHAPES + ((64, 256), (64, 256)))
        B = _log_int(rng, 1, 256)
        dtype, taps = rng.choice(DTYPES), rng.choice((1, 1, 2))
        if kind == "gen":
            T = _log_int(rng, 48, 4000)
            T = max(16, min(T, 40000 // (B + 9), 80000 // l))
            c = _net("", "gen", l, r, s, B, T, dtype, taps,
                     chunk=rng.choice((0, 0, max(16, T // 3))),
                     rule=rng.choice(("direct", "direct", "temperature", "topk")))
        else:
            T = _log_int(rng, 48, 16000)
            T = max(16, min(T, 96000 // B, 32000000 // (B * l * r)))
            c = _net("", "tf", l, r, s, B, T, dtype, taps)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _weights(c, seed):
    """fp32 host weights: matrices N(0, 1/fan_in), small biases, and an output bias that favours the
    codes around silence, as a trained voice's distributions do (a few tens of likely classes)."""
    g = torch.Generator()
    g.manual_seed(int(seed) * 2 + 1)
    l, r, s = c["l"], c["r"], c["s"]

    def mat(shape, fan_in):
        return (torch.randn(shape, generator=g) / math.sqrt(fan_in)).numpy()

    def bias(shape):
        return (0.1 * torch.randn(shape, generator=g)).numpy()

    k = np.arange(A, dtype=np.float32) - 128.0
    emb = (A, r) if c["taps"] == 1 else (2, A, r)
    return {"embed": mat(emb, c["taps"]), "b_embed": bias((r,)),
            "w_prev": mat((l, 2 * r, r), 2 * r), "w_cur": mat((l, 2 * r, r), 2 * r), "b_gate": bias((l, 2 * r)),
            "w_res": mat((l, r, r), r), "b_res": bias((l, r)),
            "w_skip": mat((l, s, r), l * r), "b_skip": bias((s,)),
            "w_relu": mat((A, s), s), "b_relu": bias((A,)),
            "w_out": mat((A, A), A), "b_out": np.maximum(-k * k / 32.0, -20.0).astype(np.float32) + bias((A,))}


def _dilations(c):
    return [1 << (i % c["cycle"]) for i in range(c["l"])]


def _audio(c, seed, T):
    """Codes of recorded audio."""
    return torch.randint(0, A, (c["B"], T), generator=_gen(seed * 7 + 3), device=DEV, dtype=torch.int32)


def _net_inputs(c, seed):
    B, T = c["B"], c["T"]
    extra = 1 if c["kind"] == "gen" else 0
    d = {"cond": torch.randn((B, T, c["l"], 2 * c["r"]), generator=_gen(seed * 7), device=DEV)}
    if extra:
        d["u"] = torch.rand((B, T), generator=_gen(seed * 7 + 1), device=DEV)
        d["cond1"] = torch.randn((B, 1, c["l"], 2 * c["r"]), generator=_gen(seed * 7 + 2), device=DEV)
        d["y"] = _audio(c, seed, 1)
    else:
        d["y"] = _audio(c, seed, T)
    return d


def _sampler(c):
    return {"direct": None, "temperature": (wn.SAMPLE_TEMPERATURE, 0.8, 0),
            "topk": (wn.SAMPLE_TOPK, 1.0, 40)}[c["rule"]]


def _cond_weights(c, seed):
    g = torch.Generator()
    g.manual_seed(int(seed) * 2 + 1)
    w = {}
    for n, h, cin in (("1", H1, FEATURES), ("2", c["l"] * c["r"], 2 * H1)):
        w["w" + n] = (torch.randn((2, 3 * h, 2, cin), generator=g) / math.sqrt(2 * cin)).numpy()
        w["b" + n] = (0.1 * torch.randn((2, 3 * h), generator=g)).numpy()
    return w


def _features(c, seed):
    """Five phonemes in context (40-way identity and 5-way stress one-hots), a voiced flag and log F0,
    phonemes of 20 frames."""
    B, F = c["B"], c["frames"]
    g = _gen(seed * 7)
    n = F // 20 + 6
    ids = torch.randint(0, 40, (B, n), generator=g, device=DEV)
    stress = torch.randint(0, 3, (B, n), generator=g, device=DEV)
    voiced = (torch.rand((B, n), generator=g, device=DEV) < 0.6).float()
    at = torch.arange(F, device=DEV) // 20
    x = torch.zeros((B, F, FEATURES), device=DEV)
    for k in range(5):
        x.scatter_(2, (40 * k + ids[:, at + k])[..., None], 1.0)
        x.scatter_(2, (200 + 5 * k + stress[:, at + k])[..., None], 1.0)
    x[..., 225] = voiced[:, at + 2]
    x[..., 226] = voiced[:, at + 2] * (2 * torch.rand((B, F), generator=g, device=DEV) - 1)
    return x


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "cond":
        net = wn.Conditioner(_cond_weights(c, seed), c["l"], c["r"], FRAME_HZ, c["audio_hz"])
        T = c["frames"] * c["audio_hz"] // FRAME_HZ
        s = {"c": c, "net": net, "x": _features(c, seed), "T": T,
             "out": torch.empty((c["B"], T, c["l"], 2 * c["r"]), device=DEV)}
        if not c["static"]:
            s["ws"] = torch.empty(net.workspace_bytes(c["B"], c["frames"]), dtype=torch.uint8, device=DEV)
        return s
    net = wn.WaveNet(_weights(c, seed), _dilations(c), weight_dtype=c["dtype"])
    s = {"c": c, "net": net, "ws": net.new_workspace(c["B"]), "sampler": _sampler(c), **_net_inputs(c, seed)}
    if c["kind"] == "tf":
        s["logits"] = torch.empty((c["B"], c["T"], A), device=DEV)
        return s
    s["logits"] = torch.empty((c["B"], 1, A), device=DEV)
    n = c["chunk"] or c["T"]
    s["parts"] = []  # inputs and outputs of the calls, one tensor each, as they come in and go out
    for a in range(0, c["T"], n):
        cond = s["cond"][:, a:a + n].contiguous()
        s["parts"].append((cond, s["u"][:, a:a + n].contiguous(),
                           torch.empty((c["B"], cond.shape[1]), dtype=torch.int32, device=DEV)))
    del s["cond"], s["u"]
    return s


def run(state):
    s, net = state, state["net"]
    kind = s["c"]["kind"]
    if kind == "cond":
        if s["c"]["static"]:
            return net.condition_static(s["x"], s["T"], s["out"])
        return net(s["x"], s["T"], cond=s["out"], workspace=s["ws"])
    if kind == "tf":
        return net.teacher_force(s["cond"], s["y"], logits=s["logits"], workspace=s["ws"])
    reset = True
    for cond, u, y in s["parts"]:
        net.generate(cond, u, samples=y, workspace=s["ws"], reset=reset, sampler=s["sampler"])
        reset = False
    net.teacher_force(s["cond1"], s["y"], logits=s["logits"], workspace=s["ws"], reset=False)
    return {"samples": [y for _, _, y in s["parts"]], "logits": s["logits"]}


def work(case):
    c = case
    if c["kind"] == "cond":
        h2, T = c["l"] * c["r"], c["frames"] * c["audio_hz"] // FRAME_HZ
        w = 2 * 3 * H1 * 2 * FEATURES + 2 * 3 * h2 * 2 * 2 * H1
        return {"bytes": 4.0 * (w + c["B"] * (c["frames"] * FEATURES + T * 2 * h2)),
                "flops": 2.0 * w * c["B"] * c["frames"]}
    l, r, s = c["l"], c["r"], c["s"]
    steps = c["B"] * (c["T"] + (1 if c["kind"] == "gen" else 0))
    mac = l * 4 * r * r + (l - 1) * r * r + l * s * r + A * s + A * A
    size = {"f32": 4, "bf16": 2, "i8": 1}[c["dtype"]]
    out = 8 if c["kind"] == "gen" else 4 + 4 * A
    return {"bytes": float(size * (mac + c["taps"] * A * r) + steps * (4 * l * 2 * r + out)),
            "flops": 2.0 * mac * steps}


def tolerance(case):
    """About four times the distance from ``exact`` (two orders of the sums, measured: fp32 and int8 models
    5.5e-8 rel and 2.1e-7 max, models on bf16 matrix products 9.2e-8 and 5.8e-7, the conditioning
    network 3.4e-7 and 3.6e-6).  A draw whose uniform falls on a rounding of the CDF may go either way
    (none in 192000 draws between two kernels)."""
    if case["kind"] == "cond":
        return {"rel": 1.5e-6, "max": 1.5e-5}
    if case["dtype"] == "f32":
        return {"rel": 2.5e-7, "max": 1.0e-6, "differ": 0.002}
    return {"rel": 4e-7, "max": 2.5e-6, "differ": 0.002}


# ------------------------------------------------------------------------------------------------
# the same outputs in 64 bits
# ------------------------------------------------------------------------------------------------
def _stored(w, dtype):
    """A matrix as the library's storage rules keep it, in fp64 on the GPU."""
    t = torch.from_numpy(np.ascontiguousarray(w))
    if dtype == "bf16":
        t = t.to(torch.bfloat16)
    elif dtype == "i8":
        d = t.double()
        sc = (d.abs().amax(-1, keepdim=True) / 127.0).float().double()
        code = torch.where(sc > 0, torch.round(d / torch.where(sc > 0, sc, torch.ones_like(sc))), torch.zeros_like(d))
        return (code.clamp(-127, 127) * sc).to(DEV)
    return t.double().to(DEV)


def _model64(c, seed):
    w = _weights(c, seed)
    mats = ("embed", "w_prev", "w_cur", "w_res", "w_skip", "w_relu", "w_out")
    m = {k: _stored(v, c["dtype"] if k in mats else "f32") for k, v in w.items()}
    if c["taps"] == 1:
        m["embed"] = m["embed"][None]
    return m


def _head64(m, q):
    z = torch.relu(torch.relu(q) @ m["w_relu"].T + m["b_relu"])
    return z @ m["w_out"].T + m["b_out"]


def _x0(m, y1, y2, has2):
    x = m["embed"][-1][y1] + m["b_embed"]
    if m["embed"].shape[0] == 2:
        x = x + m["embed"][0][y2] * has2
    return x


def _gate64(a, r):
    return torch.tanh(a[..., :r]) * torch.sigmoid(a[..., r:])


def _force64(c, m, cond, y):
    """Teacher forcing over whole sequences: each layer is a width-2 dilated causal convolution."""
    B, T, r = c["B"], c["T"], c["r"]
    y = y.long()
    first = torch.full((B, 1), 128, device=DEV)
    y1 = torch.cat([first, y[:, :-1]], 1)
    y2 = torch.cat([first, first, y[:, :-2]], 1)[:, :T]
    # y_{t-2} does not exist at the first step, and is the initial sample at the second
    has2 = (torch.arange(T, device=DEV) >= 1).double()[None, :, None]
    out = torch.empty((B, T, A), dtype=torch.float64, device=DEV)
    n = max(1, min(B, 24000 // T))
    for b in range(0, B, n):
        x = _x0(m, y1[b:b + n], y2[b:b + n], has2)
        q = m["b_skip"].expand(x.shape[0], T, -1).clone()
        for j, d in enumerate(_dilations(c)):
            back = torch.zeros_like(x)
            if d < T:
                back[:, d:] = x[:, :-d]
            h = _gate64(back @ m["w_prev"][j].T + x @ m["w_cur"][j].T + m["b_gate"][j] + cond[b:b + n, :, j].double(), r)
            q += h @ m["w_skip"][j].T
            x = x + h @ m["w_res"][j].T + m["b_res"][j]
        out[b:b + n] = _head64(m, q)
    return out


def _generate64(c, m, d):
    B, T, r = c["B"], c["T"], c["r"]
    dil = _dilations(c)
    hist = [torch.zeros((n, B, r), dtype=torch.float64, device=DEV) for n in dil]
    y1 = torch.full((B,), 128, device=DEV)
    y2, u = y1.clone(), d["u"].double()
    two = torch.cat([m["w_prev"], m["w_cur"]], 2).transpose(1, 2).contiguous()
    res, skip = m["w_res"].transpose(1, 2).contiguous(), m["w_skip"].transpose(1, 2).contiguous()
    for t in range(T + 1):
        cond = (d["cond"][:, t] if t < T else d["cond1"][:, 0]).double() + m["b_gate"]
        x, q = _x0(m, y1, y2, 1.0 if t else 0.0), m["b_skip"]
        for j, n in enumerate(dil):
            slot = hist[j][t % n]
            h = _gate64(torch.cat([slot, x], 1) @ two[j] + cond[:, j], r)
            slot.copy_(x)
            q = q + h @ skip[j]
            x = x + h @ res[j] + m["b_res"][j]
        logits = _head64(m, q)
        if t == T:
            return logits[:, None]
        e = logits / 0.8 if c["rule"] == "temperature" else logits
        if c["rule"] == "topk":
            e = e.masked_fill(e < e.topk(40, 1).values[:, -1:], -math.inf)
        cdf = torch.softmax(e, 1).cumsum(1)
        y2, y1 = y1, (cdf[:, :A - 1] <= u[:, t, None]).sum(1)


def _cond64(c, seed):
    w = {k: torch.from_numpy(v).double().to(DEV) for k, v in _cond_weights(c, seed).items()}
    x = _features(c, seed).double()
    B, F, T = c["B"], c["frames"], c["frames"] * c["audio_hz"] // FRAME_HZ
    for n, h in (("1", H1), ("2", c["l"] * c["r"])):
        dirs = []
        for k in range(2):
            z = x.flip(1) if k else x
            back = torch.cat([torch.zeros_like(z[:, :1]), z[:, :-1]], 1)
            a = back @ w["w" + n][k, :, 0].T + z @ w["w" + n][k, :, 1].T + w["b" + n][k]
            f = torch.sigmoid(a[..., 2 * h:])
            v = (1 - f) * torch.tanh(a[..., :h])
            state, hs = torch.zeros((B, h), dtype=torch.float64, device=DEV), torch.empty_like(v)
            for t in range(F):
                state = f[:, t] * state + v[:, t]
                hs[:, t] = state
            o = torch.sigmoid(a[..., h:2 * h]) * hs
            dirs.append(o.flip(1) if k else o)
        x = torch.cat(dirs, 2) if n == "1" else torch.stack(dirs, 3).reshape(B, F, 2 * h)
    at = torch.arange(T, device=DEV) * FRAME_HZ // c["audio_hz"]
    return x[:, at].reshape(B, T, c["l"], 2 * c["r"])


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "cond":
        return _cond64(c, seed)
    m, d = _model64(c, seed), _net_inputs(c, seed)
    if c["kind"] == "tf":
        return _force64(c, m, d["cond"], d["y"])
    if c["T"] * c["l"] > 100000:
        return None  # tens of seconds of small kernels
    n = len(range(0, c["T"], c["chunk"] or c["T"]))
    return {"samples": [None] * n, "logits": _generate64(c, m, d)}
