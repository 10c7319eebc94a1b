"""Teacher forcing of every step at once (the default handle's teacher_force) against the CPU oracle, and
against the step-by-step kernels, whose histories it continues and leaves.

Each case runs a call from zero at the sizes where the tiling turns: one launch for calls of up to 16
steps (several streams per 16-row tile), whole passes beyond (a partial last tile, rows of several
streams in one tile, dilations longer than the call, than a tile and of 1), on every history layout
(fp32 words, tagged words, bf16 pairs, the MFMA kernel's tiles).  Logits: every product and sum is fp32,
so their error against the 64-bit oracle is that of fp32 sums of up to l r terms of order 1 (measured
up to 2e-6; int8 and bf16 models on exact weights alike); the bound is 1e-5.  The batched kernel's histories
hold two bf16 parts of a value (2^-17 of it, times sums over r = 64 of weights of 1/sqrt(2 r), over
l layers): 1e-4.
"""
import time
import zlib

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # name, L, dilations, r, s, B, T, dtype, taps, approx, kernel family of the state
    ("stream_tiny", 4, (1, 2, 4, 8), 16, 32, 3, 17, "f32", 1, False, "stream_l2"),
    ("stream_tiny_bf16", 4, (1, 2, 4, 8), 16, 32, 5, 100, "bf16", 2, False, "stream_l2"),
    ("stream_tiny_i8_t16", 3, (3, 1, 40), 16, 32, 2, 16, "i8", 1, False, "stream_l2"),
    ("stream_l64_t5_b7", 64, tuple(synth.dilation_cycle(64)), 16, 32, 7, 5, "f32", 2, True, "stream_l2"),
    ("stream_l1_t1", 1, (1,), 16, 32, 33, 1, "bf16", 1, False, "stream_l2"),
    ("chain_r32", 5, (1, 3, 9, 27, 81), 32, 128, 2, 333, "f32", 1, False, "multi_cu_chain"),
    ("chain_r64_s128", 6, (1, 2, 4, 8, 16, 64), 64, 128, 1, 65, "f32", 1, True, "multi_cu_chain"),
    ("chain_l20", 20, tuple(synth.dilation_cycle(20)), 64, 256, 1, 1300, "f32", 2, False, "multi_cu_chain"),
    ("chain_l20_t15_b3", 20, tuple(synth.dilation_cycle(20)), 64, 256, 3, 15, "f32", 1, False, "multi_cu_chain"),
    ("chain_r128", 7, (1, 2, 4, 8, 16, 32, 64), 128, 256, 3, 50, "f32", 1, False, "multi_cu_chain"),
    ("chain_r128_t5_b7", 4, (1, 7, 2, 3), 128, 256, 7, 5, "f32", 2, True, "multi_cu_chain"),
    ("chain_bf16_b2", 6, (1, 2, 4, 8, 16, 32), 64, 256, 2, 90, "bf16", 1, False, "multi_cu_chain"),
    ("mfma_b37", 8, (1, 2, 4, 8, 16, 32, 64, 128), 64, 256, 170, 40, "bf16", 1, False, "multi_cu_mfma"),
    ("mfma_i8_t1", 8, (1, 2, 4, 8, 16, 32, 64, 128), 64, 256, 170, 1, "i8", 2, False, "multi_cu_mfma"),
    # 16 streams per replica, one per tile column (WN_MFMA_COLUMNS), fewer in the last
    ("mfma_16_columns", 5, (1, 2, 4, 8, 16), 64, 256, 67, 30, "bf16", 1, False, "multi_cu_mfma"),
    ("mfma_16_columns_t3", 5, (1, 2, 4, 8, 16), 64, 256, 67, 3, "i8", 1, False, "multi_cu_mfma"),
    ("group_s128", 5, (1, 2, 4, 8, 16), 64, 128, 150, 25, "bf16", 1, False, "mfma_group"),
]


def _sequence(net, cond, u, y, cuts):
    """Generation, teacher forcing in the given pieces, then generation, all on one state."""
    ws = net.new_workspace(cond.shape[0])
    n = u.shape[1] // 2
    first = net.generate(cond[:, :n].contiguous(), u[:, :n].contiguous(), workspace=ws)
    lg, a = [], 0
    for b in cuts:
        lg.append(net.teacher_force(cond[:, n + a:n + b].contiguous(), y[:, a:b].contiguous(), workspace=ws, reset=False))
        a = b
    last = net.generate(cond[:, n + a:].contiguous(), u[:, n:].contiguous(), workspace=ws, reset=False)
    assert net.status(ws) == 0
    return first, torch.cat(lg, 1), last


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_teacher_forcing_parallel(case, monkeypatch):
    import paper_1702_07825_amd as wn
    name, L, dil, r, s, B, T, dtype, taps, approx, family = case
    print("teacher forcing %s: L=%d r=%d s=%d B=%d T=%d %s" % (name, L, r, s, B, T, dtype), flush=True)
    seed = zlib.crc32(name.encode()) % 1000
    if name.startswith("mfma_16_columns"):
        monkeypatch.setenv("WN_MFMA_COLUMNS", "16")
    w = synth.make_weights(L, r, s, seed=seed, bias_scale=0.2, embed_taps=taps)
    net = wn.WaveNet(w, dil, weight_dtype=dtype, approx_nonlin=approx)
    assert net.kernel_variant(B) == family
    monkeypatch.setenv("WN_KERNEL", "stream" if family == "stream_l2" else family)
    step = wn.WaveNet(w, dil, weight_dtype=dtype, approx_nonlin=approx)  # step by step
    monkeypatch.delenv("WN_KERNEL")
    assert step.kernel_variant(B) == family
    bound = 1e-4 if family in ("mfma_group", "multi_cu_mfma") else 1e-5
    cond = synth.make_cond(L, r, B, T + 10, seed=seed, device="cuda")
    u = torch.tensor(synth.make_uniforms(B, 10, seed=seed), device="cuda")
    y = torch.tensor(synth.make_samples(B, T, seed=seed), device="cuda")

    lg = net.teacher_force(cond[:, :T].contiguous(), y)
    mode = {"bf16": {"bf16_weights": True}, "i8": {"int8_weights": True}}.get(dtype, {})
    model = oracle.Model(w, dil, approx_nonlin=approx, **mode)
    some = sorted({0, B // 2, B - 1})
    _, lo, _ = oracle.run_streams(model, cond[some, :T].cpu().numpy(), y_in=y[some].cpu().numpy(), threads=3)
    err = float(np.abs(lg[some].cpu().numpy() - lo).max())
    print("  max|dlogit| oracle %.3g" % err, flush=True)
    assert err <= (1e-4 if family == "mfma_group" else 1e-5)

    # on a state that generation left, in one call and cut where the two forms meet: the same logits
    # bit for bit, within the step kernels' own error of theirs, and a state they continue alike
    f0, l0, g0 = _sequence(net, cond, u, y, (T,))
    f1, l1, g1 = _sequence(net, cond, u, y, tuple(sorted({1, min(T, 16), min(T, 17), T})))
    f2, l2, g2 = _sequence(step, cond, u, y, (T,))
    assert torch.equal(f0, f1) and torch.equal(f0, f2)
    assert torch.equal(l0, l1) and torch.equal(g0, g1)
    assert float((l0 - l2).abs().max()) <= 2 * bound
    # draws part where a uniform lies within that error of a CDF value: at most a few streams of a batch
    assert float((g0 != g2).any(1).float().mean()) <= (0.0 if B < 8 else 0.05)

    # generation after a prompt forced from zero: as from the state the step kernel leaves, up to the same margin
    after = []
    for k in (net, step):
        ws = k.new_workspace(B)
        k.teacher_force(cond[:, :T].contiguous(), y, workspace=ws)
        after.append(k.generate(cond[:, T:].contiguous(), u, workspace=ws, reset=False))
        assert k.status(ws) == 0
    assert float((after[0] != after[1]).any(1).float().mean()) <= (0.0 if B < 8 else 0.05)

    # a workspace without the scratch serves the call step by step
    ws = net.new_workspace(B)
    small = ws[:step.workspace_bytes(B)]
    assert torch.equal(net.teacher_force(cond[:, :T].contiguous(), y, workspace=small),
                       step.teacher_force(cond[:, :T].contiguous(), y))

    # a standing abort request: nothing is written
    net.abort(True)
    out = torch.full((B, T, 256), -1.0, device="cuda")
    net.teacher_force(cond[:, :T].contiguous(), y, logits=out, workspace=ws)
    assert net.status(ws) == wn.WN_EABORTED and bool((out == -1.0).all())
    net.abort(False)
    assert torch.equal(net.teacher_force(cond[:, :T].contiguous(), y, workspace=ws), lg) and net.status(ws) == 0
    net.close()
    step.close()


TALL = [
    # name, L, dilations, r, s, B, T, approx: rows just past where the tiles of a pass grow from 16 to 32 rows, and
    # at r = 128 to 48 (one block per CU there: half the tiles)
    ("r32", 3, (1, 40, 7), 32, 128, 1, 8193, False),
    ("r64_s128", 3, (1, 33, 600), 64, 128, 2, 4100, False),
    ("r64_s128_approx", 3, (1, 33, 600), 64, 128, 3, 2750, True),
    ("r64", 3, (5, 1, 64), 64, 256, 1, 8193, False),
    ("r128_32", 3, (1, 2, 100), 128, 256, 1, 4097, False),
    ("r128_48", 3, (1, 2, 100), 128, 256, 1, 8193, False),
    ("r128_48_approx", 2, (50, 1), 128, 256, 5, 1700, True),
]


@pytest.mark.parametrize("case", TALL, ids=[c[0] for c in TALL])
def test_tall_tiles(case):
    """The builds of a pass with tiles of 32 and 48 rows: against the oracle (bound as above), and bit for bit the
    logits of calls short enough for tiles of 16."""
    import paper_1702_07825_amd as wn
    name, L, dil, r, s, B, T, approx = case
    print("tall tiles %s" % name, flush=True)
    w = synth.make_weights(L, r, s, seed=14, bias_scale=0.2)
    net = wn.WaveNet(w, dil, approx_nonlin=approx)
    cond = synth.make_cond(L, r, B, T, seed=14, device="cuda")
    y = torch.tensor(synth.make_samples(B, T, seed=14), device="cuda")
    lg = net.teacher_force(cond, y)
    model = oracle.Model(w, dil, approx_nonlin=approx)
    _, lo, _ = oracle.run_streams(model, cond.cpu().numpy(), y_in=y.cpu().numpy(), threads=5)
    err = float(np.abs(lg.cpu().numpy() - lo).max())
    print("  max|dlogit| oracle %.3g" % err, flush=True)
    assert err <= 1e-5
    ws, parts, n = net.new_workspace(B), [], 2048 // B
    for a in range(0, T, n):
        parts.append(net.teacher_force(cond[:, a:a + n].contiguous(), y[:, a:a + n].contiguous(), workspace=ws, reset=a == 0))
    assert torch.equal(torch.cat(parts, 1), lg) and net.status(ws) == 0
    net.close()


@pytest.mark.parametrize("B", [1536, 1537])
def test_short_calls_of_many_small_streams(B):
    """r = 16: up to 512 tiles (of 3 streams at 5 steps) go in one launch, one more stream in a pass: the same logits
    bit for bit, from zero and continued, as calls of a few of the streams."""
    import paper_1702_07825_amd as wn
    L, T = 3, 5
    net = wn.WaveNet(synth.make_weights(L, 16, 32, seed=17, bias_scale=0.2), (1, 4, 9))
    print("short calls, B=%d" % B, flush=True)
    cond = synth.make_cond(L, 16, B, 2 * T, seed=17, device="cuda")
    y = torch.tensor(synth.make_samples(B, 2 * T, seed=17), device="cuda")

    def two(some):
        c, yy, ws = cond[some].contiguous(), y[some].contiguous(), net.new_workspace(len(some))
        out = [net.teacher_force(c[:, a:a + T].contiguous(), yy[:, a:a + T].contiguous(), workspace=ws, reset=a == 0)
               for a in (0, T)]
        assert net.status(ws) == 0
        return torch.cat(out, 1)
    whole, some = two(list(range(B))), [0, 1, 2, 3, B // 2, B - 2, B - 1]
    assert torch.equal(whole[some], two(some))
    net.close()


def test_chunks_of_a_long_call():
    """More rows than the scratch holds: chunks over steps and over streams give the same logits as calls
    that fit (4 layers, so that the sizes stay small)."""
    import paper_1702_07825_amd as wn
    w = synth.make_weights(4, 16, 32, seed=3, bias_scale=0.2)
    net = wn.WaveNet(w, (1, 5, 300, 2))
    for B, T in ((1, 40000), (200, 403)):
        print("chunks: B=%d T=%d" % (B, T), flush=True)
        cond = synth.make_cond(4, 16, B, T, seed=4, device="cuda")
        y = torch.tensor(synth.make_samples(B, T, seed=4), device="cuda")
        whole = net.teacher_force(cond, y)
        parts = [net.teacher_force(cond[b:b + 1, :1500].contiguous(), y[b:b + 1, :1500].contiguous()) for b in (0, B - 1)]
        assert torch.equal(whole[0, :1500], parts[0][0]) and torch.equal(whole[B - 1, :1500], parts[1][0])
        ws = net.new_workspace(B)
        h = T // 2 + 1
        a = net.teacher_force(cond[:, :h].contiguous(), y[:, :h].contiguous(), workspace=ws)
        b = net.teacher_force(cond[:, h:].contiguous(), y[:, h:].contiguous(), workspace=ws, reset=False)
        assert torch.equal(torch.cat([a, b], 1), whole)
    net.close()


def test_timeout_path_drains_and_recovers(monkeypatch):
    """The waits between tiles are bounded: with the host's spin limit forced to one poll a call of many tiles ends
    with WN_ETIMEOUT (every block leaves, so the stream drains), and the next call from zero on the same
    workspace gives the logits of an undisturbed one."""
    import paper_1702_07825_amd as wn
    L, r, s, B, T = 20, 64, 256, 2, 8000  # 500 tiles, two to a CU
    net = wn.WaveNet(synth.make_weights(L, r, s, seed=9, bias_scale=0.1), tuple(synth.dilation_cycle(L)))
    cond = synth.make_cond(L, r, B, T, seed=9, device="cuda")
    y = torch.tensor(synth.make_samples(B, T, seed=9), device="cuda")
    ws = net.new_workspace(B)
    ref = net.teacher_force(cond, y)
    monkeypatch.setenv("WN_SPIN_LIMIT", "1")
    print("teacher forcing: forced timeout", flush=True)
    net.teacher_force(cond, y, workspace=ws)
    assert net.status(ws) == wn.WN_ETIMEOUT
    monkeypatch.delenv("WN_SPIN_LIMIT")
    assert torch.equal(net.teacher_force(cond, y, workspace=ws, reset=True), ref) and net.status(ws) == 0
    net.close()


def test_abort_between_the_chunks_of_a_call():
    """A request made while a call of many chunks runs ends it at a chunk: the steps of the later ones are not
    written, and the next call from zero on the same workspace is undisturbed."""
    import paper_1702_07825_amd as wn
    L, r, s, B, T = 20, 64, 256, 4, 150000
    net = wn.WaveNet(synth.make_weights(L, r, s, seed=15, bias_scale=0.1), tuple(synth.dilation_cycle(L)))
    cond = torch.zeros((B, T, L, 2 * r), device="cuda")
    y = torch.tensor(synth.make_samples(B, 3000, seed=15), device="cuda").repeat(1, T // 3000)
    ws = net.new_workspace(B)
    ref = net.teacher_force(cond[:, :500].contiguous(), y[:, :500].contiguous())
    out = torch.empty((B, T, 256), device="cuda")
    net.teacher_force(cond, y, logits=out, workspace=ws)
    assert net.status(ws) == 0
    t0 = time.perf_counter()
    net.teacher_force(cond, y, logits=out, workspace=ws)
    assert net.status(ws) == 0
    full = time.perf_counter() - t0
    out.fill_(-1.0)
    torch.cuda.synchronize()
    net.teacher_force(cond, y, logits=out, workspace=ws)
    time.sleep(0.2 * full)
    net.abort(True)
    status = net.status(ws)
    net.abort(False)
    written = (out[0, :, 0] != -1.0).sum().item()
    print("  a whole call takes %.1f ms; aborted after %d of %d steps" % (1e3 * full, written, T), flush=True)
    assert status == wn.WN_EABORTED
    assert bool((out[:, -1] == -1.0).all())
    again = net.teacher_force(cond[:, :500].contiguous(), y[:, :500].contiguous(), workspace=ws, reset=True)
    assert torch.equal(again, ref) and net.status(ws) == 0
    net.close()


def test_waits_while_another_stream_holds_compute_units(monkeypatch):
    """A long kernel of another stream (192 workgroups, each filling a CU) keeps most of a call's 512 tiles off the chip
    for many times the spin limit.  With a dilation of 256 tiles each tile that runs waits for one that does not:
    the call finishes once all have run, and its logits are those of a call alone."""
    import paper_1702_07825_amd as wn
    L, r, s, T = 4, 16, 32, 16384
    dil = (8192, 1, 2, 4)
    w = synth.make_weights(L, r, s, seed=10, bias_scale=0.2)
    net, other = wn.WaveNet(w, dil), wn.WaveNet(w, (1, 2, 4, 8))
    assert net.kernel_variant(1) == "stream_l2"
    cond = synth.make_cond(L, r, 1, T, seed=10, device="cuda")
    y = torch.tensor(synth.make_samples(1, T, seed=10), device="cuda")
    ref = net.teacher_force(cond, y)
    BG, TG = 192, 16000
    busy_cond = torch.zeros((BG, TG, L, 2 * r), device="cuda")
    busy_u = torch.rand((BG, TG), device="cuda")
    busy_ws, ws = other.new_workspace(BG), net.new_workspace(1)
    out = torch.full((1, T, 256), -1.0, device="cuda")
    side = torch.cuda.Stream()
    other.generate(busy_cond[:, :100].contiguous(), busy_u[:, :100].contiguous(), workspace=busy_ws, stream=side)
    torch.cuda.synchronize()
    monkeypatch.setenv("WN_SPIN_LIMIT", "2000")  # about 2 ms of polls
    print("teacher forcing beside a kernel that holds 192 CUs", flush=True)
    t0 = time.perf_counter()
    busy_y = other.generate(busy_cond, busy_u, workspace=busy_ws, stream=side)
    time.sleep(0.004)  # it runs by now
    net.teacher_force(cond, y, logits=out, workspace=ws)
    status = net.status(ws)
    took = time.perf_counter() - t0
    assert other.status(busy_ws, stream=side) == 0
    print("  status %d after %.1f ms, the other kernel's call took %.1f" % (status, 1e3 * took, 1e3 * (time.perf_counter() - t0)),
          flush=True)
    assert status == 0 and torch.equal(out, ref)
    assert torch.equal(net.teacher_force(cond, y, workspace=ws, reset=True), ref) and net.status(ws) == 0
    assert int(busy_y.min()) >= 0 and int(busy_y.max()) <= 255
    net.close()
    other.close()


@pytest.mark.parametrize("B", [1099, 1100])
def test_batches_that_the_batched_kernel_forces_itself(B, monkeypatch):
    """From 1100 streams on the batched kernel is the faster one and takes teacher forcing step by step, whatever a
    call's length, in a workspace without the scratch; one stream fewer takes all steps of a call at once."""
    import paper_1702_07825_amd as wn
    L, r, s, T = 2, 64, 128, 18
    w = synth.make_weights(L, r, s, seed=12, bias_scale=0.2)
    net = wn.WaveNet(w, (1, 3), weight_dtype="bf16")
    monkeypatch.setenv("WN_KERNEL", "mfma_group")
    step = wn.WaveNet(w, (1, 3), weight_dtype="bf16")
    monkeypatch.delenv("WN_KERNEL")
    print("batched kernel's line, B=%d" % B, flush=True)
    assert net.kernel_variant(B) == step.kernel_variant(B) == "mfma_group"
    cond = synth.make_cond(L, r, B, T, seed=12, device="cuda")
    y = torch.tensor(synth.make_samples(B, T, seed=12), device="cuda")
    lg, ls = net.teacher_force(cond, y), step.teacher_force(cond, y)
    own = B >= 1100
    assert (net.workspace_bytes(B) == step.workspace_bytes(B)) == own and torch.equal(lg, ls) == own
    assert float((lg - ls).abs().max()) <= 1e-4
    ws = net.new_workspace(B)
    parts = [net.teacher_force(cond[:, a:b].contiguous(), y[:, a:b].contiguous(), workspace=ws, reset=a == 0)
             for a, b in ((0, 1), (1, T))]
    assert torch.equal(torch.cat(parts, 1), lg) and net.status(ws) == 0
    net.close()
    step.close()
