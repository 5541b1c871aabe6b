"""GPU parity of the backward path and of recurrent decoding against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import act64, dev_act, dev_f32, host, params_dev, params_np, rel_err, say, tol

pytestmark = pytest.mark.gpu

ops = None
GRADS = ("dgamma", "domega", "damp", "dphase")


def setup_module(module):
    global ops
    from paper_2607_05583_amd import ops as _ops
    ops = _ops
    assert torch.cuda.is_available(), "GPU tests need a HIP device"


def _check_bwd(prob, act, use_h0, bound_dx, bound_p):
    x = dev_act(prob["x"], act)
    dy = dev_act(prob["dy"], act)
    h0 = dev_f32(prob["h0"]) if use_h0 else None
    g = ops.resonator_mix_bwd(x, dy, *params_dev(prob), h0=h0, want_dh0=True)
    torch.cuda.synchronize()
    ref = O.mix_bwd(act64(prob["x"], act), act64(prob["dy"], act), *params_np(prob),
                    h0=prob["h0"] if use_h0 else None)
    errs = {"dx": rel_err(host(g["dx"]), ref["dx"])}
    for k in GRADS:
        errs[k] = rel_err(host(g[k]), ref[k])
    errs["dh0"] = rel_err(host(g["dh0"]), ref["dh0"])
    say("  errs " + " ".join(f"{k}={v:.2e}" for k, v in errs.items()))
    assert errs["dx"] <= bound_dx
    for k in (*GRADS, "dh0"):
        assert errs[k] <= bound_p, k
    return g


BWD_SMALL = [
    (1, 1, 1, 1, False, 31),
    (2, 15, 3, 2, True, 32),
    (1, 300, 33, 8, True, 33),
    (2, 513, 64, 5, False, 34),
    (3, 777, 70, 16, True, 35),
    (1, 2048, 32, 8, False, 36),
]


@pytest.mark.parametrize("B,L,D,M,use_h0,seed", BWD_SMALL)
@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_bwd_small_shapes(B, L, D, M, use_h0, seed, act):
    say(f"bwd small B={B} L={L} D={D} M={M} h0={use_h0} {act}")
    prob = W.random_problem(seed, B, L, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True,
                            with_h0=use_h0, with_dy=True)
    if act == "f32":
        _check_bwd(prob, act, use_h0, 1e-4, 1e-4)
    else:
        _check_bwd(prob, act, use_h0, 2e-2, 2e-2)


# Segment geometries of the backward (a row of P tiles in nseg segments of S
# tiles, about one work-group per compute unit): a ragged last segment with a
# partial last tile, one multi-tile segment per row (no segment records), and
# short segments with two mode groups, ragged D and h0.
BWD_SEGMENTS = [
    (8, 9372, 256, 8, "bf16", True, 37),
    (8, 9372, 256, 8, "f32", False, 38),
    (32, 1024, 256, 8, "bf16", False, 39),
    (3, 5000, 96, 12, "f32", True, 40),
    # float32 with an even segment length: records per half segment; a partial
    # last tile, and a last record segment shorter than the others
    (4, 8000, 256, 8, "f32", True, 41),
    (4, 7580, 256, 8, "f32", False, 42),
]


def _segments(B, L, D, act):
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    dw = 32 if act == "bf16" else 16
    chains, P = B * ((D + dw - 1) // dw), (L + 255) // 256
    nseg = max(1, min(P, ncu // chains if ncu > chains else 1))
    S = -(-P // nseg)
    nseg = -(-P // S)
    return nseg, S, P - (nseg - 1) * S


def _record_segments(M, act, S):
    """Record segments per segment of the segment pass (float32, one mode group,
    an even segment length: two)."""
    return 2 if act == "f32" and M <= 8 and S % 2 == 0 else 1


@pytest.mark.parametrize("B,L,D,M,act,use_h0,seed", BWD_SEGMENTS)
def test_bwd_segment_geometries(B, L, D, M, act, use_h0, seed):
    nseg, S, last = _segments(B, L, D, act)
    sf = _record_segments(M, act, S)
    say(f"bwd segments B={B} L={L} D={D} M={M} {act} h0={use_h0}: {nseg} segments of {S} tiles (last {last}), "
        f"records per {S // sf} tiles")
    prob = W.random_problem(seed, B, L, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True,
                            with_h0=use_h0, with_dy=True)
    tol = 1e-4 if act == "f32" else 2e-2
    _check_bwd(prob, act, use_h0, tol, tol)


def test_bwd_deterministic():
    say("bwd determinism")
    prob = W.random_problem(40, 2, 3000, 64, 8, act="bf16", gamma_range=(1e-4, 1.0), gamma_log=True,
                            with_dy=True)
    x, dy = dev_act(prob["x"], "bf16"), dev_act(prob["dy"], "bf16")
    pr = params_dev(prob)
    a = ops.resonator_mix_bwd(x, dy, *pr)
    b = ops.resonator_mix_bwd(x, dy, *pr)
    torch.cuda.synchronize()
    for k in ("dx", *GRADS):
        assert torch.equal(a[k], b[k]), k


def test_autograd_function_matches_bwd():
    say("autograd wrapper")
    prob = W.random_problem(41, 2, 300, 32, 4, act="f32", with_dy=True)
    x = dev_act(prob["x"], "f32").requires_grad_(True)
    pr = [p.clone().requires_grad_(True) for p in params_dev(prob)]
    y = ops.resonator_mix(x, *pr)
    y.backward(dev_act(prob["dy"], "f32"))
    ref = O.mix_bwd(prob["x"], prob["dy"], *params_np(prob))
    assert rel_err(host(x.grad), ref["dx"]) <= 1e-4
    for p, k in zip(pr, GRADS):
        assert rel_err(host(p.grad), ref[k]) <= 1e-4


@pytest.mark.parametrize("layer", range(6))
def test_config5_training_layer(layer):
    """Training config: each of the 6 layers fwd + bwd at B8 L8192 D256 M8, bf16 activations."""
    cfg = W.CONFIGS[5]
    say(f"config 5 layer {layer}")
    inp = W.train_layer_inputs(cfg, layer)
    x = dev_act(inp["x"], "bf16")
    pr = params_dev(inp)
    y = ops.resonator_mix_fwd(x, *pr)
    torch.cuda.synchronize()
    x64 = act64(inp["x"], "bf16")
    yr = O.mix_recurrence(x64, *params_np(inp))[0]
    ey = rel_err(host(y), yr)
    say(f"  y err {ey:.2e}")
    assert ey <= 2e-2
    _check_bwd(inp, "bf16", False, 2e-2, 2e-2)


# --------------------------------------------------------------------------
# decode
# --------------------------------------------------------------------------
@pytest.mark.parametrize("B,D,M,L0,steps,seed", [(1, 1, 1, 0, 5, 51), (3, 7, 3, 10, 40, 52),
                                                 (64, 256, 8, 300, 200, 53), (5, 70, 16, 1, 64, 54)])
@pytest.mark.parametrize("act,out", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
def test_decode_small(B, D, M, L0, steps, seed, act, out):
    say(f"decode small B={B} D={D} M={M} L0={L0} steps={steps} {act}->{out}")
    prob = W.random_problem(seed, B, L0 + steps, D, M, act=act, gamma_range=(1e-4, 1.0),
                            gamma_log=True)
    x = dev_act(prob["x"], act)
    pr = params_dev(prob)
    st = ops.resonator_state_init(x[:, :L0].contiguous(), *pr)
    ys = []
    for t in range(L0, L0 + steps):
        ys.append(ops.resonator_decode_step(x[:, t].contiguous(), *pr, st,
                                            out_dtype=torch.float32 if out == "f32" else x.dtype))
    torch.cuda.synchronize()
    yg = np.stack([host(v) for v in ys], 1)
    x64 = act64(prob["x"], act)
    yr, hr = O.mix_recurrence(x64, *params_np(prob))
    assert rel_err(yg, yr[:, L0:]) <= tol(act, out)
    assert rel_err(host(st), hr) <= (1e-4 if act == "f32" else 2e-2)


@pytest.mark.parametrize("B,D,M,L0,steps,seed", [(1, 1, 1, 0, 1, 61), (3, 7, 3, 10, 40, 62),
                                                 (64, 256, 8, 300, 200, 63), (5, 70, 16, 1, 64, 64),
                                                 (9, 130, 5, 0, 33, 65)])
@pytest.mark.parametrize("act,out", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
def test_decode_steps(B, D, M, L0, steps, seed, act, out):
    """N steps in one launch: bitwise the same outputs and state as N single decode
    steps, and within the decode tolerance of the oracle recurrence."""
    say(f"decode steps B={B} D={D} M={M} L0={L0} steps={steps} {act}->{out}")
    prob = W.random_problem(seed, B, L0 + steps, D, M, act=act, gamma_range=(1e-4, 1.0),
                            gamma_log=True)
    x = dev_act(prob["x"], act)
    pr = params_dev(prob)
    od = torch.float32 if out == "f32" else x.dtype
    st1 = ops.resonator_state_init(x[:, :L0].contiguous(), *pr)
    st2 = st1.clone()
    ys = [ops.resonator_decode_step(x[:, t].contiguous(), *pr, st1, out_dtype=od)
          for t in range(L0, L0 + steps)]
    yn = ops.resonator_decode_steps(x[:, L0:].contiguous(), *pr, st2, out_dtype=od)
    torch.cuda.synchronize()
    assert torch.equal(torch.stack(ys, 1), yn)
    assert torch.equal(st1, st2)
    yr, hr = O.mix_recurrence(act64(prob["x"], act), *params_np(prob))
    assert rel_err(host(yn), yr[:, L0:]) <= tol(act, out)
    assert rel_err(host(st2), hr) <= (1e-4 if act == "f32" else 2e-2)


@pytest.mark.parametrize("B,D,M,K,act", [(3, 70, 5, 16, "bf16"), (64, 256, 8, 64, "bf16"), (2, 33, 16, 7, "f32")])
def test_decode_graph_replays_match_eager_steps(B, D, M, K, act):
    """A captured K-step decode loop, replayed three times with new drives (eager
    work and synchronisations between the replays), gives bitwise the outputs and
    state of K eager decode steps every time."""
    say(f"decode graph B={B} D={D} M={M} K={K} {act}")
    prob = W.random_problem(92 + K, B, 20 + 3 * K, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True)
    x = dev_act(prob["x"], act)
    pr = params_dev(prob)
    st_g = ops.resonator_state_init(x[:, :20].contiguous(), *pr)
    st_e = st_g.clone()
    g = ops.DecodeGraph(*pr, st_g, K, x_dtype=x.dtype)
    torch.cuda.synchronize()
    assert torch.equal(st_g, st_e)  # capture runs nothing
    for r in range(3):
        drives = x[:, 20 + r * K:20 + (r + 1) * K].transpose(0, 1).contiguous()  # [K, B, D]
        ye = torch.stack([ops.resonator_decode_step(drives[k], *pr, st_e) for k in range(K)])
        torch.cuda.synchronize()
        yg = g.replay(drives)
        torch.cuda.synchronize()
        assert torch.equal(yg, ye), r
        assert torch.equal(st_g, st_e), r
        _ = (x.float() * 2).sum().item()  # unrelated eager work between the replays


@pytest.mark.parametrize("B,D,M,N,act", [(1, 1, 1, 8, "f32"), (5, 65, 8, 7, "bf16"), (5, 63, 9, 17, "bf16"),
                                         (256, 256, 2, 9, "f32"), (257, 256, 3, 9, "bf16"), (1024, 65, 9, 3, "f32")])
def test_decode_steps_kernel_choice(B, D, M, N, act):
    """Both kernels of several steps (a lane per mode up to 65536 (b, d) pairs, a
    thread per pair above), on batch-major and time-major drives and at the
    remainders of the lanes' step batches: bitwise N single steps."""
    say(f"decode steps kernels B={B} D={D} M={M} N={N} {act}")
    prob = W.random_problem(171 + B, B, N, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True, with_h0=True)
    x, pr = dev_act(prob["x"], act), params_dev(prob)
    st0 = torch.from_numpy(prob["h0"]).cuda()
    st1, st2, st3 = st0.clone(), st0.clone(), st0.clone()
    ye = torch.stack([ops.resonator_decode_step(x[:, t].contiguous(), *pr, st1) for t in range(N)], 1)
    yn = ops.resonator_decode_steps(x, *pr, st2)
    yg = ops.DecodeGraph(*pr, st3, N, x_dtype=x.dtype).replay(x.transpose(0, 1).contiguous())
    torch.cuda.synchronize()
    assert torch.equal(yn, ye) and torch.equal(st2, st1)
    assert torch.equal(yg, ye.transpose(0, 1)) and torch.equal(st3, st1)


@pytest.mark.parametrize("B,D,M,N,act", [(512, 256, 8, 1, "bf16"), (1024, 65, 16, 1, "f32"), (1030, 64, 1, 2, "bf16"),
                                         (4096, 16, 4, 3, "bf16"), (4096, 16, 8, 33, "f32"), (2000, 16, 10, 5, "bf16"),
                                         (700, 9, 3, 11, "f32"), (129, 500, 12, 20, "bf16")])
def test_decode_steps_kernel_rule(B, D, M, N, act):
    """Both sides of the rule between a lane per mode and a thread per pair, narrow
    inputs (small groups of channel blocks) and one step of many pairs: bitwise N
    single steps."""
    test_decode_steps_kernel_choice(B, D, M, N, act)


@pytest.mark.parametrize("B,D,M", [(262144, 1, 1), (300001, 2, 9)])
def test_decode_graph_of_many_rows(B, D, M):
    """More batch rows than a grid's second dimension holds in blocks of four:
    bitwise the single steps."""
    say(f"decode graph B={B} D={D} M={M}")
    g = torch.Generator(device="cuda").manual_seed(B)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    pr = [r(D, M).abs() + 1e-3, r(D, M), r(D, M), r(D, M)]
    x, st0 = r(3, B, D), r(B, D, M, 2)
    st1, st2 = st0.clone(), st0.clone()
    want = torch.stack([ops.resonator_decode_step(x[t], *pr, st1) for t in range(3)])
    got = ops.DecodeGraph(*pr, st2, 3, x_dtype=torch.float32).replay(x)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(st2, st1)


def _oracle_rows(args):
    """Oracle recurrence over one group of batch rows (a worker thread's share)."""
    x, h0, prm = args
    return O.mix_recurrence(x, *prm, h0=h0)


def test_config4_decode_full():
    """Decode config: prompt 1024 -> state_init, then 32768 decode steps at B64 D256 M8 (bf16).

    Every output of every batch row and the final state are compared with the
    oracle's recurrence (Sec. 3.3) started from the oracle's prompt state; the
    oracle runs chunk by chunk over eight groups of rows in worker threads.
    """
    from concurrent.futures import ThreadPoolExecutor

    cfg = W.CONFIGS[4]
    say(f"config 4 {cfg.name}")
    di = W.DecodeInputs(cfg)
    pr = params_dev(di.params)
    prm = params_np(di.params)
    prompt = dev_act(di.prompt, "bf16")
    st = ops.resonator_state_init(prompt, *pr)
    torch.cuda.synchronize()
    st_ref = O.state_init(act64(di.prompt, "bf16"), *prm)
    assert rel_err(host(st), st_ref) <= 2e-2
    n_total, chunk = cfg.steps, 4096
    groups = [slice(g, g + 8) for g in range(0, cfg.B, 8)]
    h = [st_ref[g] for g in groups]
    worst = 0.0
    y_dev = torch.empty((chunk, cfg.B, cfg.D), dtype=torch.bfloat16, device="cuda")
    with ThreadPoolExecutor(max_workers=8) as pool:
        for s0 in range(0, n_total, chunk):
            xs = di.steps(chunk)  # [chunk, B, D]
            xd = dev_act(xs, "bf16")
            for j in range(chunk):
                ops.resonator_decode_step(xd[j], *pr, st, out=y_dev[j])
            x64 = np.ascontiguousarray(act64(xs, "bf16").transpose(1, 0, 2))  # [B, chunk, D]
            res = list(pool.map(_oracle_rows, [(x64[g], h[i], prm) for i, g in enumerate(groups)]))
            torch.cuda.synchronize()
            yg = host(y_dev).transpose(1, 0, 2)  # [B, chunk, D]
            yr = np.concatenate([r[0] for r in res], 0)
            h = [r[1] for r in res]
            worst = max(worst, rel_err(yg, yr))
            say(f"  steps {s0 + chunk}: worst step err so far {worst:.3e}")
    say(f"config 4 worst step err {worst:.3e}")
    assert worst <= 2e-2
    assert rel_err(host(st), np.concatenate(h, 0)) <= 2e-2


@pytest.mark.parametrize("single", [False, True])
def test_decode_long_f32_within_1e4(single):
    """32768 float32 decode steps (slow modes down to gamma = 1e-5) stay within the
    float32 bound of the oracle recurrence on every output and on the final
    state: the pole is applied as a float32 hi + lo pair, so the phase error of a
    single rounded pole does not build up over the run.  Drives come in blocks
    of 2048 steps per launch (resonator_decode_steps, bitwise single steps) or,
    for one block, as single steps."""
    B, D, M, steps, blk = 2, 24, 8, 32768, 2048
    say(f"decode long f32 B={B} D={D} M={M} steps={steps} single={single}")
    prob = W.random_problem(301, B, steps, D, M, act="f32", gamma_range=(1e-5, 1.0), gamma_log=True,
                            with_h0=True)
    x = dev_act(prob["x"], "f32")
    pr = params_dev(prob)
    st = dev_f32(prob["h0"])
    ys = []
    for s0 in range(0, steps, blk):
        if single and s0 == steps - blk:
            ys.append(torch.stack([ops.resonator_decode_step(x[:, t].contiguous(), *pr, st)
                                   for t in range(s0, s0 + blk)], 1))
        else:
            ys.append(ops.resonator_decode_steps(x[:, s0:s0 + blk].contiguous(), *pr, st))
    torch.cuda.synchronize()
    yg = host(torch.cat(ys, 1))
    yr, hr = O.mix_recurrence(prob["x"], *params_np(prob), h0=prob["h0"])
    e, eh = rel_err(yg, yr), rel_err(host(st), hr)
    say(f"  rel err y {e:.3e} state {eh:.3e}")
    assert e <= 1e-4
    assert eh <= 1e-4


@pytest.mark.parametrize("B,D,M,act,out,shift", [(64, 256, 8, "bf16", "bf16", False), (5, 70, 5, "f32", "f32", False),
                                                 (3, 33, 16, "bf16", "f32", False), (17, 40, 8, "f32", "f32", True)])
def test_decode_step_from_table_is_bitwise_the_step(B, D, M, act, out, shift):
    """Decode from the constants table (one evaluation of the constants, then
    table-driven steps) gives bitwise the outputs and state of resonator_decode_step
    over 12 steps, with the table 16-byte aligned (the fast path) or only 8-byte
    aligned (shift); and it follows the oracle's recurrence."""
    say(f"decode from table B={B} D={D} M={M} {act}->{out} shift={shift}")
    prob = W.random_problem(71 + M, B, 40, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True)
    x = dev_act(prob["x"], act)
    pr = params_dev(prob)
    od = torch.float32 if out == "f32" else torch.bfloat16
    st1 = ops.resonator_state_init(x[:, :28].contiguous(), *pr)
    st2 = st1.clone()
    if shift:
        buf = torch.empty(D * M * 6 + 2, dtype=torch.float32, device="cuda")
        tab = ops.resonator_decode_constants(*pr, out=buf[2:].view(D, M, 6))
    else:
        tab = ops.resonator_decode_constants(*pr)
    ys = []
    for k in range(28, 40):
        xk = x[:, k].contiguous()
        y1 = ops.resonator_decode_step(xk, *pr, st1, out_dtype=od)
        y2 = ops.resonator_decode_step_tab(xk, tab, st2, out_dtype=od)
        torch.cuda.synchronize()
        assert torch.equal(y1, y2), k
        assert torch.equal(st1, st2), k
        ys.append(y2)
    yr, hr = O.mix_recurrence(act64(prob["x"], act), *params_np(prob))
    assert rel_err(host(torch.stack(ys, 1)), yr[:, 28:]) <= tol(act, out)
    assert rel_err(host(st2), hr) <= (1e-4 if act == "f32" else 2e-2)
