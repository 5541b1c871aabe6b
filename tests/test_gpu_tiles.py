"""Edges of the tiled kernels against the float64 oracle: prompt states over several
segments and partial first tiles, forwards whose tiles are not full (16-byte
pieces inside and outside the tensor, rows that are no pieces), mode banks past
one group.

Tolerances: float32 sums of up to a few thousand terms with float64-built powers
stay under 1e-4 (rel_err: over the larger of |value| and rms), bf16 outputs
round to 2^-9, and bf16 tables are split to 2^-17 (2e-2 is the suite's gate)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import act64, dev_act, dev_f32, host, params_dev, params_np, rel_err, say, tol

pytestmark = pytest.mark.gpu


def _prob(seed, B, L, D, M, act, **kw):
    return W.random_problem(seed, B, L, D, M, act=act, gamma_range=(1e-4, 1.0), gamma_log=True, **kw)


@pytest.mark.parametrize("B,L,D,M", [(1, 5000, 40, 16), (1, 70000, 16, 3), (2, 4099, 24, 8), (300, 300, 8, 2),
                                     (1, 2561, 33, 9), (3, 256, 64, 1)])
@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_prompt_state_segments(B, L, D, M, act):
    from paper_2607_05583_amd import ops
    say(f"prompt state B={B} L={L} D={D} M={M} {act}")
    prob = _prob(L, B, L, D, M, act)
    st = ops.resonator_state_init(dev_act(prob["x"], act), *params_dev(prob))
    ref = O.state_init(act64(prob["x"], act), *params_np(prob))
    assert rel_err(host(st), ref) <= (1e-4 if act == "f32" else 2e-2)
    # bf16 drives are exact and the split tables carry 16 bits: the state is closer than the outputs
    assert np.linalg.norm(host(st) - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("B,L,D,M", [(1, 257, 8, 8), (2, 300, 200, 6), (3, 769, 72, 8), (1, 511, 264, 4),
                                     (2, 700, 65, 8), (1, 4100, 136, 12), (2, 1030, 24, 16), (1, 3000, 31, 10),
                                     (260, 520, 8, 16)])
@pytest.mark.parametrize("act,out", [("f32", "f32"), ("bf16", "bf16"), ("bf16", "f32")])
def test_forward_partial_tiles(B, L, D, M, act, out):
    from paper_2607_05583_amd import ops
    say(f"forward B={B} L={L} D={D} M={M} {act}->{out}")
    prob = _prob(L + D, B, L, D, M, act, with_h0=True)
    y, h = ops.resonator_mix_fwd(dev_act(prob["x"], act), *params_dev(prob), h0=dev_f32(prob["h0"]),
                                 out_dtype=torch.float32 if out == "f32" else torch.bfloat16, return_state=True)
    yr, hr = O.mix_recurrence(act64(prob["x"], act), *params_np(prob), h0=prob["h0"])
    assert rel_err(host(y), yr) <= tol(act, out)
    assert rel_err(host(h), hr) <= (1e-4 if act == "f32" else 2e-2)


@pytest.mark.parametrize("L,D,M", [(16, 64, 8), (16, 24, 16), (11, 65, 3), (300, 64, 8), (4096, 40, 16)])
@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_prompt_state_keeps_float32_bits(L, D, M, act):
    """Drives only in the last 16 steps (one chunk, nothing to damp an error).  Powers
    rounded once to float32 and float32 sums of 16 terms: each rounding is at most
    2^-24 of the sum of the terms' magnitudes, 17 of them (two-part bf16 powers are
    2^-17 off)."""
    from paper_2607_05583_amd import ops
    say(f"prompt state bits L={L} D={D} M={M} {act}")
    prob = _prob(L + D, 2, L, D, M, act)
    prob["x"][:, :max(L - 16, 0)] = 0
    st = host(ops.resonator_state_init(dev_act(prob["x"], act), *params_dev(prob)))
    x, p = act64(prob["x"], act), params_np(prob)
    ref = O.state_init(x, *p)
    lim = O.state_init(np.abs(x), p[0], np.zeros_like(p[1]), *p[2:])[..., :1]  # sum of |lambda|^k |x|
    assert np.all(np.abs(st - ref) <= 17 * 2.0 ** -24 * lim + 1e-30)


@pytest.mark.parametrize("B,L,D,M", [(8, 33000, 64, 9), (1, 33024, 24, 12), (1, 131328, 16, 16)])
@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_forward_long_rows_wide_bank(B, L, D, M, act):
    """Carry fold past 128 tiles a row: segments of 16 tiles (many rows, or more than
    512 tiles) and of 4 tiles doubled."""
    from paper_2607_05583_amd import ops
    say(f"forward long rows B={B} L={L} D={D} M={M} {act}")
    prob = _prob(L + M, B, L, D, M, act, with_h0=True)
    y, h = ops.resonator_mix_fwd(dev_act(prob["x"], act), *params_dev(prob), h0=dev_f32(prob["h0"]), return_state=True)
    rows = [0, B - 1] if B > 1 else [0]
    x = act64(prob["x"], act)
    yr, hr = O.mix_recurrence(x[rows], *params_np(prob), h0=prob["h0"][rows])
    assert rel_err(host(y)[rows], yr) <= tol(act, act)
    assert rel_err(host(h)[rows], hr) <= (1e-4 if act == "f32" else 2e-2)
