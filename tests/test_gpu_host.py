"""The native marshalling of the hot calls against the Python marshalling of the
same calls (the native module switched off), and the workspace a call makes for
itself: bitwise equal, on allocations that hold other data."""
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu


class _Off:
    """Stands in for the native module: takes nothing, so the Python code runs."""

    def __getattr__(self, name):
        return lambda *a: None


@pytest.fixture
def ops(monkeypatch):
    from paper_2607_05583_amd import ops as _ops
    monkeypatch.setattr(_ops, "CHECK_FWD_STATUS", False)
    monkeypatch.setattr(_ops, "_NATIVE", _ops._native())
    return _ops


def _params(D, M, g):
    r = lambda: torch.rand(D, M, device="cuda", generator=g)
    return [r() * 0.5 + 1e-3, r() * 3, torch.randn(D, M, device="cuda", generator=g), r() * 6]


def _flat(o):
    if isinstance(o, torch.Tensor):
        return [o]
    if isinstance(o, dict):
        o = [o[k] for k in sorted(o)]
    return [t for e in o if e is not None for t in _flat(e)]


def _both(monkeypatch, ops, call):
    # memory the allocator hands out again: words with the tag of a first call, and all ones
    got = []
    for word in (1 << 32, -1):
        torch.cuda.empty_cache()
        junk = torch.full((8 << 20,), word, dtype=torch.int64, device="cuda")
        small = [torch.full((1 << 16,), word, dtype=torch.int64, device="cuda") for _ in range(16)]
        del junk, small
        got.append(_flat(call()))
    monkeypatch.setattr(ops, "_NATIVE", _Off())
    b = _flat(call())
    for a in got:
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert x.shape == y.shape and x.dtype == y.dtype and torch.equal(x, y)


@pytest.mark.parametrize("B,L,D,M", [(1, 40, 8, 1), (2, 3000, 72, 8), (3, 1030, 65, 6), (2, 700, 64, 12)])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("what", ["fwd", "bwd", "state", "steps", "step"])
def test_mixing_calls(monkeypatch, ops, what, dt, B, L, D, M):
    say(f"native {what} B={B} L={L} D={D} M={M} {dt}")
    g = torch.Generator(device="cuda").manual_seed(L + M)
    prm, x = _params(D, M, g), torch.randn(B, L, D, device="cuda", generator=g).to(dt)
    h0 = torch.randn(B, D, M, 2, device="cuda", generator=g)
    calls = {
        "fwd": lambda: ops.resonator_mix_fwd(x, *prm, h0=h0, return_state=True, out_dtype=torch.float32),
        "bwd": lambda: ops.resonator_mix_bwd(x, x, *prm, h0=h0, want_dh0=True),
        "state": lambda: ops.resonator_state_init(x, *prm),
        "steps": lambda: (ops.resonator_decode_steps(x[:, :20].contiguous(), *prm, h := h0.clone()), h),
        "step": lambda: (ops.resonator_decode_step(x[:, 0].contiguous(), *prm, h := h0.clone()), h),
    }
    _both(monkeypatch, ops, calls[what])


@pytest.mark.parametrize("dt,dh,K", [(torch.bfloat16, 32, 4), (torch.float32, 16, 3), (torch.float32, 24, 0)])
@pytest.mark.parametrize("save", [False, True])
def test_block_calls(monkeypatch, ops, dt, dh, K, save):
    H, B, L, M = 4, 2, 333, 8
    D = H * dh
    say(f"native block {dt} dh={dh} K={K} save={save}")
    g = torch.Generator(device="cuda").manual_seed(dh)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    x, W = r(B, L, D).to(dt), [(r(H, dh, dh) / dh ** 0.5).to(dt) for _ in range(3)]
    w, s = (r(D, K), r(D)) if K else (None, None)
    args = (x, *W, *_params(D, M, g), r(H, H), 0.5, w, s, H)

    def call():
        out, saved = ops.resonator_block_fwd(*args, save=True) if save else (ops.resonator_block_fwd(*args), None)
        return out, ops.resonator_block_bwd(*args, out, saved=saved)

    _both(monkeypatch, ops, call)


def test_refusals_keep_their_messages(ops):
    x, prm = torch.randn(1, 8, 4, device="cuda"), [torch.rand(4, 2, device="cuda") for _ in range(4)]
    with pytest.raises(ValueError, match="contiguous"):
        ops.resonator_mix_fwd(x.transpose(1, 2), *prm)
    with pytest.raises(ValueError, match="D=4"):
        ops.resonator_mix_fwd(torch.randn(1, 8, 5, device="cuda"), *prm)
    with pytest.raises(KeyError):
        ops.resonator_mix_fwd(x.half(), *prm)
    with pytest.raises(ValueError, match="workspace too small"):
        ops.resonator_mix_fwd(x, *prm, ws=torch.zeros(16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(Exception, match="overlap"):
        ops.resonator_mix_fwd(x, *prm, out=x)
    with pytest.raises(ValueError, match="state must be"):
        ops.resonator_decode_steps(x, *prm, torch.zeros(1, 4, 3, 2, device="cuda"))


def test_outputs_that_are_too_small_are_refused(ops):
    """A given output smaller than what the call writes raises before any launch; a
    larger one takes the result in its first elements."""
    B, L, D, M, H = 2, 40, 32, 3, 2
    g = torch.Generator(device="cuda").manual_seed(9)
    prm, x = _params(D, M, g), torch.randn(B, L, D, device="cuda", generator=g)
    W = torch.randn(H, D // H, D // H, device="cuda", generator=g)
    h, Ct = torch.zeros(B, D, M, 2, device="cuda"), torch.zeros(H, H, device="cuda")
    calls = {
        "mix": (B * L * D, lambda o: ops.resonator_mix_fwd(x, *prm, out=o)),
        "state": (B * D * M * 2, lambda o: ops.resonator_state_init(x, *prm, out=o)),
        "step": (B * D, lambda o: ops.resonator_decode_step(x[:, 0].contiguous(), *prm, h, out=o)),
        "step_tab": (B * D, lambda o: ops.resonator_decode_step_tab(
            x[:, 0].contiguous(), ops.resonator_decode_constants(*prm), h, out=o)),
        "steps": (B * L * D, lambda o: ops.resonator_decode_steps(x, *prm, h, out=o)),
        "linear": (B * L * D, lambda o: ops.resonator_grouped_linear(x, W, out=o)),
        "linear2": (B * L * D, lambda o: ops.resonator_grouped_linear2(x, W, W, out0=o, out1=o.clone())),
        "extract": (D * D // H, lambda o: ops.resonator_block_diag_extract(torch.ones(D, D, device="cuda"), H, out=o)),
        "epilogue": (B * L * D, lambda o: ops.resonator_epilogue_fwd(x, x, None, Ct, 0.5, None, None, H, out=o)),
        "epilogue_proj": (B * L * D, lambda o: ops.resonator_epilogue_proj_fwd(x, x, None, Ct, 0.5, None, None, H, W,
                                                                              out=o)),
    }
    for name, (n, call) in calls.items():
        say(f"given output {name}")
        with pytest.raises(ValueError, match="too small"):
            call(torch.empty(n - 1, device="cuda"))
        h.zero_()
        exact, larger = torch.empty(n, device="cuda"), torch.full((n + 64,), 7.0, device="cuda")
        call(exact)
        h.zero_()
        call(larger)
        assert torch.equal(larger[:n], exact) and bool((larger[n:] == 7.0).all())
    with pytest.raises(ValueError, match="must be torch.float32"):
        ops.resonator_state_init(x, *prm, out=torch.empty(B, D, M, 2, device="cuda", dtype=torch.bfloat16))
    with pytest.raises(ValueError, match="on the GPU"):
        ops.resonator_decode_step(x[:, 0].contiguous(), *prm, h, out=torch.empty(B, D))


@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs two GPUs")
def test_calls_run_on_their_tensors_gpu(ops):
    """Calls and replays on the second GPU while the first is current (their default
    streams are both the null stream, which means the current device)."""
    g = torch.Generator(device="cuda:0").manual_seed(4)
    prm, x = _params(40, 6, g), torch.randn(3, 500, 40, device="cuda:0", generator=g)
    h = torch.randn(3, 40, 6, 2, device="cuda:0", generator=g)
    outs = []
    for dev in ("cuda:0", "cuda:1"):
        p, xd, hd = [t.to(dev) for t in prm], x.to(dev), h.to(dev)
        graph = ops.DecodeGraph(*p, hd, 5, x_dtype=torch.float32)
        torch.cuda.synchronize(dev)
        with torch.cuda.device(0):
            r = [ops.resonator_mix_fwd(xd, *p), ops.resonator_state_init(xd, *p),
                 graph.replay(xd[:, :5].transpose(0, 1).contiguous()), hd]
        torch.cuda.synchronize(dev)
        outs.append([t.cpu() for t in r])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("native", [True, False])
def test_decode_replay_under_capture(monkeypatch, ops, native):
    """A replay launches the graph's kernel itself: eagerly, recorded into a caller's
    capture, and the same as the graph's own work, by either marshalling."""
    g = torch.Generator(device="cuda").manual_seed(3)
    prm, B, N, D, M = _params(24, 5, g), 3, 7, 24, 5
    x, s0 = torch.randn(N, B, D, device="cuda", generator=g), torch.randn(B, D, M, 2, device="cuda", generator=g)
    live, ref = s0.clone(), s0.clone()
    graph = ops.DecodeGraph(*prm, live, N, x_dtype=x.dtype)
    if not native:
        monkeypatch.setattr(ops, "_NATIVE", _Off())

    def want():
        return ops.resonator_decode_steps(x.transpose(0, 1).contiguous(), *prm, ref).transpose(0, 1)

    for _ in range(3):
        y = graph.replay(x)
        w = want()
        torch.cuda.synchronize()
        assert torch.equal(y, w) and torch.equal(live, ref)
    graph.graph.replay()
    assert torch.equal(graph.y, want()) and torch.equal(live, ref)
    static = x.clone()
    outer = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(outer):
        y = graph.replay(static)
        twice = y * 2
    assert torch.equal(live, ref)  # recorded, not run
    for i in range(4):
        x = torch.randn(N, B, D, device="cuda", generator=g)
        static.copy_(x)
        outer.replay()
        w = want()
        torch.cuda.synchronize()
        assert torch.equal(graph.y, w) and torch.equal(twice, w * 2) and torch.equal(live, ref)
        _ = (x * i).sum().item()  # eager work between the replays


@pytest.mark.parametrize("dt,dh", [(torch.bfloat16, 32), (torch.float32, 16)])
def test_block_graph_with_the_calls_own_workspace(ops, dt, dh):
    """A captured block: its forward clears the words it uses of a workspace of its
    own inside the capture.  Replays against eager calls, with eager work between."""
    H, B, L, M, K = 4, 2, 1500, 8, 3
    D = H * dh
    say(f"block graph {dt} dh={dh}")
    g = torch.Generator(device="cuda").manual_seed(dh + 1)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    W = [(r(H, dh, dh) / dh ** 0.5).to(dt) for _ in range(3)]
    args = (*W, *_params(D, M, g), r(H, H), 0.5, r(D, K), r(D), H)
    graph = ops.BlockForwardGraph(r(B, L, D).to(dt), *args)
    for i in range(4):
        x = r(B, L, D).to(dt)
        want = ops.resonator_block_fwd(x, *args)
        torch.cuda.synchronize()
        got = graph.replay(x)
        torch.cuda.synchronize()
        assert torch.equal(got, want), i
        _ = (x.float() * i).sum().item()


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("keep", [False, True])
def test_forward_past_4096_chains(ops, dt, keep):
    """Chains 4096 .. use the second group of counter words; twice on one workspace.
    Every row is the same problem, so the first row's float64 recurrence checks all."""
    B, L, D, M = 9000, 40, 8, 5
    say(f"forward chains={B} {dt} keep={keep}")
    g = torch.Generator(device="cuda").manual_seed(8)
    prm = _params(D, M, g)
    row = torch.randn(1, L, D, device="cuda", generator=g).to(dt)
    x, ws = row.expand(B, L, D).contiguous(), ops.forward_workspace(dt, B, L, D, M, "cuda") if keep else None
    gam, om, amp, ph = (p.double().cpu() for p in prm)
    lam = torch.exp(torch.complex(-gam, om))
    h, want = torch.zeros(D, M, dtype=torch.complex128), []
    for t in range(L):
        h = lam * h + row[0, t].double().cpu()[:, None]
        want.append((amp * torch.exp(1j * ph) * h).real.sum(-1))
    want = torch.stack(want)
    for _ in range(2):
        y = ops.resonator_mix_fwd(x, *prm, ws=ws, out_dtype=torch.float32)
        assert bool((y == y[:1]).all())
        err = (y[0].double().cpu() - want).norm() / want.norm()
        # float32 sums of some tens of terms; bf16 drives are exact, their tables 2^-17
        assert err <= (1e-6 if dt == torch.float32 else 2.0 ** -15)
        if keep:
            assert ops.resonator_fwd_status(ws) == 0
