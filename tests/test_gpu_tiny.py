"""Generation with the smallest models (r = 16, s = 32, weights resident on one CU per stream) against the CPU
oracle and the per-stream kernel, whose state it shares.

Sample indices must be the oracle's wherever its CDF margin (the rule's own margin for the others) exceeds
1e-4, as for every kernel; both kernels sum in fp32, so their samples part only at a margin below that.
Cases: one and the most layers it takes (8; with 9 the per-stream kernel serves), dilations of 1, 2 and
longer than the call, a batch, two taps, each weight format, calls split at odd steps and across the
64-step staging of the uniforms, each sampling rule, the approximate nonlinearities."""
import time
import zlib

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MARGIN = 1e-4
CASES = [
    # name, L, dilations, B, T, dtype, taps, approx, sampler (wn_sampler: mode, temperature, top_k)
    ("l4", 4, (1, 2, 4, 8), 1, 200, "f32", 1, False, None),
    ("l1_d1_t1", 1, (1,), 3, 1, "f32", 1, False, None),
    ("l8_b5_2tap", 8, (1, 2, 1, 300, 3, 2, 64, 1), 5, 133, "f32", 2, False, None),
    ("l9_stream", 9, (1, 2, 4, 8, 1, 2, 4, 8, 1), 2, 70, "f32", 1, False, None),
    ("l3_bf16", 3, (2, 1, 5), 2, 130, "bf16", 2, False, (1, 0.7, 0)),
    ("l6_i8", 6, (1, 2, 4, 8, 16, 32), 2, 129, "i8", 1, False, (2, 1.0, 20)),
    ("l4_approx", 4, (1, 2, 4, 8), 2, 100, "f32", 1, True, None),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_tiny_generation(case, monkeypatch):
    import paper_1702_07825_amd as wn
    name, L, dil, B, T, dtype, taps, approx, smp = case
    print("tiny %s" % name, flush=True)
    seed = zlib.crc32(name.encode()) % 1000
    w = synth.make_weights(L, 16, 32, seed=seed, bias_scale=0.2, embed_taps=taps)
    net = wn.WaveNet(w, dil, weight_dtype=dtype, approx_nonlin=approx)
    monkeypatch.setenv("WN_KERNEL", "stream")
    ref = wn.WaveNet(w, dil, weight_dtype=dtype, approx_nonlin=approx)
    monkeypatch.delenv("WN_KERNEL")
    cond = synth.make_cond(L, 16, B, T, seed=seed, device="cuda")
    u = torch.tensor(synth.make_uniforms(B, T, seed=seed), device="cuda")
    y = net.generate(cond, u, sampler=smp)
    mode = {"bf16": {"bf16_weights": True}, "i8": {"int8_weights": True}}.get(dtype, {})
    model = oracle.Model(w, dil, approx_nonlin=approx, **mode)
    y_np = y.cpu().numpy()
    # the oracle's draws on the kernel's own samples
    kw = {} if smp is None else {"sampler": smp}
    ys, _, mg = oracle.run_streams(model, cond.cpu().numpy(), u=u.cpu().numpy(), y_in=y_np, threads=4, **kw)
    ok = mg > MARGIN
    print("  confident %d of %d, mismatches %d" % (int(ok.sum()), ok.size, int(np.sum(ys[ok] != y_np[ok]))), flush=True)
    assert np.array_equal(ys[ok], y_np[ok])
    yr = ref.generate(cond, u, sampler=smp).cpu().numpy()
    for b in range(B):
        low = np.nonzero(~ok[b])[0]
        first = int(low[0]) if low.size else T
        assert np.array_equal(y_np[b, :first], yr[b, :first])
    # calls split at odd steps, alternating with the per-stream kernel on the same state
    ws = net.new_workspace(B)
    parts, a = [], 0
    for k, e in enumerate(sorted({1, min(T, 2), min(T, 63), min(T, 66), T})):
        if e > a:
            parts.append(net.generate(cond[:, a:e].contiguous(), u[:, a:e].contiguous(), workspace=ws, reset=a == 0, sampler=smp))
        a = e
    assert net.status(ws) == 0 and torch.equal(torch.cat(parts, 1), y)
    if T > 40:  # from a state that the per-stream kernel left, as from its own
        ws, h = net.new_workspace(B), T // 2
        first = [k.generate(cond[:, :h].contiguous(), u[:, :h].contiguous(), workspace=ws[:ref.workspace_bytes(B)], sampler=smp)
                 for k in (net, ref)]
        rest = ref.generate(cond[:, h:].contiguous(), u[:, h:].contiguous(), workspace=ws[:ref.workspace_bytes(B)], reset=False, sampler=smp)
        ref.generate(cond[:, :h].contiguous(), u[:, :h].contiguous(), workspace=ws[:ref.workspace_bytes(B)], sampler=smp)
        other = net.generate(cond[:, h:].contiguous(), u[:, h:].contiguous(), workspace=ws, reset=False, sampler=smp)
        for b in range(B):
            if ok[b].all() and torch.equal(first[0][b], first[1][b]):
                assert torch.equal(rest[b], other[b])
    # a standing abort request: no step is taken; withdrawn, a call from zero is undisturbed
    net.abort(True)
    out = torch.full((B, T), -1, dtype=torch.int32, device="cuda")
    net.generate(cond, u, samples=out, workspace=ws, sampler=smp)
    assert net.status(ws) == wn.WN_EABORTED and bool((out == -1).all())
    net.abort(False)
    assert torch.equal(net.generate(cond, u, workspace=ws, sampler=smp), y) and net.status(ws) == 0
    net.close()
    ref.close()


def _kernels(call):
    """Names of the kernels that call() launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return " ".join(e.key for e in prof.key_averages())


@pytest.mark.parametrize("L,tiny", [(8, True), (9, False)])
def test_the_kernel_that_runs(L, tiny):
    """Up to 8 layers generation runs the kernel with resident weights, beyond the per-stream one (wn_kernel_variant
    names the family, and with it the state's layout, for both)."""
    import paper_1702_07825_amd as wn
    net = wn.WaveNet(synth.make_weights(L, 16, 32, seed=2), (1, 2, 4, 8, 1, 2, 4, 8, 16)[:L])
    cond = synth.make_cond(L, 16, 2, 20, seed=2, device="cuda")
    u = torch.tensor(synth.make_uniforms(2, 20, seed=2), device="cuda")
    ran = _kernels(lambda: net.generate(cond, u))
    print("  kernels: %s" % ran, flush=True)
    assert ("wn_tiny_kernel" in ran) == tiny and ("wn_stream_kernel" in ran) == (not tiny)
    net.close()


def test_abort_during_a_call():
    """A request made while a call runs stops it within 64 steps; the next call from zero is undisturbed."""
    import paper_1702_07825_amd as wn
    L, B, T = 4, 2, 200000
    net = wn.WaveNet(synth.make_weights(L, 16, 32, seed=6, bias_scale=0.1), (1, 2, 4, 8))
    cond = synth.make_cond(L, 16, B, T, seed=6, device="cuda")
    u = torch.tensor(synth.make_uniforms(B, T, seed=6), device="cuda")
    ws = net.new_workspace(B)
    ref = net.generate(cond[:, :200].contiguous(), u[:, :200].contiguous(), workspace=ws)
    t0 = time.perf_counter()
    net.generate(cond, u, workspace=ws)
    assert net.status(ws) == wn.WN_OK
    full = time.perf_counter() - t0
    y = torch.full((B, T), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    net.generate(cond, u, samples=y, workspace=ws)
    time.sleep(0.2 * full)
    net.abort(True)
    status = net.status(ws)
    took = time.perf_counter() - t0
    net.abort(False)
    print("  a whole call takes %.1f ms; aborted after %.1f" % (1e3 * full, 1e3 * took), flush=True)
    assert status == wn.WN_EABORTED and took < 0.8 * full
    taken = [int((y[b] != -1).sum()) for b in range(B)]
    assert all(n % 64 == 0 and bool((y[b, n:] == -1).all()) for b, n in enumerate(taken))
    again = net.generate(cond[:, :200].contiguous(), u[:, :200].contiguous(), workspace=ws, reset=True)
    assert torch.equal(again, ref) and net.status(ws) == wn.WN_OK
    net.close()
