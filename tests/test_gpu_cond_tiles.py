"""The conditioning network at the sizes where its kernels turn: the contraction's 128 x 128 tiles (from 512
blocks on, ragged in frames and gate rows) beside the 64 x 64 ones, the pool's passes of 128 frames in
segments of 16 (one frame more and less) and its single segments of short sequences, and an output whose rows end inside a block's run of 1024 pieces.

Against the oracle (64-bit): the split bf16 products keep fp32's precision, so a gate pre-activation of up to
1024 terms with standard deviation near 1 is off by about 1024^(1/2) x 2^-24 = 2e-6, and the outputs, bounded by
1, by a few times that (measured up to 4e-6 of their rms): 2e-5.  Features of 2^60 put the parts of a value far apart and
saturate the gates, which hold to the same bound."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # name, F, h1, n_layers, r, B, n_frames, frame_rate, audio_rate, scale of the features
    ("tiles128", 227, 256, 20, 64, 5, 221, 256, 300, 1.0),
    ("seg127", 36, 40, 2, 19, 3, 127, 3, 8, 1.0),
    ("seg128", 36, 40, 2, 19, 2, 128, 3, 8, 1.0),
    ("seg129", 36, 40, 2, 19, 2, 129, 3, 8, 1.0),
    ("seg257_wide", 64, 32, 2, 32, 1, 257, 256, 16000, 1.0),
    # short sequences: one segment of 1, 4 or 16 frames and 256 channels to a block, and the first that takes more
    ("seg1", 36, 300, 2, 19, 3, 1, 1, 3, 1.0),
    ("seg2", 36, 40, 2, 150, 2, 2, 3, 8, 1.0),
    ("seg4", 36, 40, 2, 150, 2, 4, 3, 8, 1.0),
    ("seg5", 36, 300, 2, 19, 2, 5, 3, 8, 1.0),
    ("seg16", 36, 40, 2, 150, 2, 16, 3, 8, 1.0),
    ("seg17", 36, 40, 2, 150, 2, 17, 3, 8, 1.0),
    ("saturated", 227, 48, 2, 16, 2, 40, 1, 1, 2.0 ** 60),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_conditioning_tiles(case):
    import paper_1702_07825_amd as wn
    name, F, h1, L, r, B, Tf, fr, ar, scale = case
    print("cond tiles %s" % name, flush=True)
    w = synth.make_cond_weights(F, h1, L * r, seed=len(name), bias_scale=0.2)
    x = (np.random.default_rng(7).normal(0, 1, (B, Tf, F)) * scale).astype(np.float32)
    T = (Tf * ar) // fr
    net = wn.Conditioner(w, L, r, fr, ar)
    got = net(torch.tensor(x, device="cuda"), T).cpu().numpy().reshape(B, T, 2 * L * r)
    for b in sorted({0, B - 1}):
        ref = oracle.condition(w, x[b], T, fr, ar)
        err = float(np.abs(got[b] - ref).max())
        print("  stream %d max|dcond| = %.3g" % (b, err), flush=True)
        assert err <= 2e-5
    net.close()


@pytest.mark.parametrize("F,h1,L,r,B,Tf", [(227, 48, 2, 16, 2, 40), (36, 32, 2, 32, 1, 70), (64, 256, 20, 64, 5, 221)],
                         ids=["scalar_loads", "vector_loads", "tiles128"])
def test_infinite_and_largest_values(F, h1, L, r, B, Tf):
    """Infinities and fp32's largest value, in the features and in the weights: the sum of a gate is then infinite
    or beyond 1e30 of one sign (one such term per sum), so the gates saturate and every output stays within the
    bound above.  Split into parts, such a value would meet products of both signs."""
    import paper_1702_07825_amd as wn
    rng = np.random.default_rng(11)
    top = np.finfo(np.float32).max
    x = rng.normal(0, 1, (B, Tf, F)).astype(np.float32)
    plain = synth.make_cond_weights(F, h1, L * r, seed=3, bias_scale=0.2)
    x_odd = x.copy()
    for i, t in enumerate(range(1, Tf, 3)):  # a width-2 window sees one of them
        x_odd[:, t, (5 * i) % F] = (np.inf, -np.inf, top, -top)[i % 4]
    w_odd = {k: v.copy() for k, v in plain.items()}
    for i, n in enumerate(range(0, 3 * h1, 5)):
        w_odd["w1"][i % 2, n, 1, (3 * i) % F] = (np.inf, -np.inf, top, -top)[i // 2 % 4]
    for name, w, xs in (("features", plain, x_odd), ("weights", w_odd, x)):
        net = wn.Conditioner(w, L, r, 1, 1)
        got = net(torch.tensor(xs, device="cuda"), Tf).cpu().numpy().reshape(B, Tf, 2 * L * r)
        net.close()
        for b in sorted({0, B - 1}):
            ref = oracle.condition(w, xs[b], Tf, 1, 1)
            assert np.isfinite(ref).all()
            err = float(np.abs(got[b] - ref).max())
            print("  odd %s stream %d max|dcond| = %.3g" % (name, b, err), flush=True)
            assert err <= 2e-5


@pytest.mark.parametrize("F,h1,L,r,B,Tf", [(227, 48, 2, 16, 2, 40), (36, 32, 2, 32, 1, 70), (64, 256, 20, 64, 5, 221)],
                         ids=["scalar_loads", "vector_loads", "tiles128"])
def test_products_near_the_largest_value(F, h1, L, r, B, Tf):
    """Products just below fp32's largest value (0.997 x 2^128, exact in 24 bits) whose operands round up to 2^64 as
    bf16, cancelled by two products of half the size: the sum is 0 in any order, while the bf16 parts' product alone is
    infinite (and the cancelling ones are finite, so no NaN tells)."""
    import paper_1702_07825_amd as wn
    v = np.float32(2045.0 / 1024.0 * 2.0 ** 63)
    w = synth.make_cond_weights(F, h1, L * r, seed=5, bias_scale=0.2)
    x = np.random.default_rng(13).normal(0, 1, (B, Tf, F)).astype(np.float32)
    x[:, ::3, 1:4] = v
    for c in range(0, h1, 5):  # the channel's h~ is the three terms alone; its o and f only their biases
        w["b1"][:, c] = 0.0
        for gate in range(3):
            w["w1"][:, c + gate * h1] = 0.0
        w["w1"][:, c, 1, 1:4] = (v, -v / 2, -v / 2)
    x[:, 1::3, 1:4] = x[:, 2::3, 1:4] = 0.0  # (elsewhere the three terms would saturate the gate either way)
    net = wn.Conditioner(w, L, r, 1, 1)
    got = net(torch.tensor(x, device="cuda"), Tf).cpu().numpy().reshape(B, Tf, 2 * L * r)
    net.close()
    for b in sorted({0, B - 1}):
        ref = oracle.condition(w, x[b], Tf, 1, 1)
        assert np.isfinite(ref).all()
        err = float(np.abs(got[b] - ref).max())
        print("  stream %d max|dcond| = %.3g" % (b, err), flush=True)
        assert err <= 2e-5
