"""GPU parity of the fp32 forward at the edges of its tiles (32 queries x 32 keys, key tiles dealt
to 4 or 8 waves, depth slots in chunks of 3 or 6): against the fp64 oracle, through the C ABI.

Tolerance 1e-5 (max abs): |O| <= 5 here and a weight or an output is a sum of at most a few hundred
terms rounded at 2^-24 relative, an error of some 1e-6 at most."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import moda_attn_fwd, synth
from paper_2603_15619_amd.binding import MODAShape, lib

pytestmark = pytest.mark.gpu
TOL = 1e-5


def run(B, Hq, Hk, T, d, L, seed, causal=True, depth_alloc=None, spoil=None):
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="f32", seed=seed, device="cuda", depth_alloc=depth_alloc)
    if depth_alloc is not None and depth_alloc > L:
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    ref = R.fwd(*(None if inp[k] is None else np.nan_to_num(synth.to_f64(inp[k]))
                  for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), depth_count=L, causal=causal)
    if spoil is not None:
        inp["Vseq"][:, :, spoil[0]] = spoil[1]
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"], depth_count=L,
                           causal=causal)
    torch.cuda.synchronize()
    return synth.to_f64(O), synth.to_f64(LSE), ref


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 0, None), (2, 2, 1, 31, 128, 3, 4), (1, 2, 2, 32, 64, 6, 7),
                                              (1, 3, 1, 33, 128, 4, None), (1, 4, 2, 95, 64, 7, None), (1, 2, 2, 96, 128, 0, None),
                                              (1, 8, 8, 129, 64, 1, 3), (3, 8, 2, 161, 128, 13, None), (1, 2, 1, 517, 128, 2, None)])
def test_f32_tile_edges(B, Hq, Hk, T, d, L, La, causal):
    O, LSE, (Oref, Lref) = run(B, Hq, Hk, T, d, L, 40 + T + L, causal, La)
    assert np.abs(O - Oref).max() <= TOL and np.abs(LSE - Lref).max() <= TOL


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,four", [(32, 8, 4, 9, 64, 5, 6, False), (43, 6, 3, 32, 128, 4, None, True), (33, 4, 2, 33, 64, 7, 8, True),
                                                   (22, 3, 1, 97, 128, 6, None, True), (8, 8, 2, 100, 64, 13, None, False), (13, 4, 4, 129, 128, 1, 2, True),
                                                   (2, 2, 2, 257, 128, 0, None, False), (2, 2, 2, 256, 64, 0, None, True),
                                                   (2, 4, 2, 256, 128, 1, 2, True), (2, 4, 2, 256, 128, 2, None, False), (2, 4, 4, 257, 128, 1, None, False),
                                                   (2, 4, 4, 100, 64, 1, None, False)])
def test_f32_four_and_eight_waves(B, Hq, Hk, T, d, L, La, four, causal):
    """Both sides of the line between four waves per workgroup and eight, which takes up to 256 tiles with slots (d = 128:
    two or more of them) or more than 256 positions."""
    s = MODAShape(B, Hq, Hk, T, d, L if La is None else La, L, int(causal), 0.0, 0)
    name = ctypes.create_string_buffer(64)
    lib().moda_fwd_kernel_name(ctypes.byref(s), None, name, len(name))
    assert name.value.decode() == "moda_fwd_f32_%skernel<%d>" % ("four_" if four else "", d)
    O, LSE, (Oref, Lref) = run(B, Hq, Hk, T, d, L, 140 + T + L, causal, La)
    assert np.abs(O - Oref).max() <= TOL and np.abs(LSE - Lref).max() <= TOL


@pytest.mark.parametrize("Hq,T,d,L", [(5, 2000, 128, 2), (9, 1999, 64, 0)])
def test_f32_grids_of_one_round(Hq, T, d, L):
    """Between one and three workgroups per compute unit, a number that 8 does not divide: tiles of every
    other layer in reverse."""
    O, LSE, (Oref, Lref) = run(1, Hq, Hq, T, d, L, 60 + T)
    assert np.abs(O - Oref).max() <= TOL and np.abs(LSE - Lref).max() <= TOL


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("T,d,at", [(70, 64, 37), (130, 128, 129), (64, 128, 0), (6, 64, 3)])
def test_f32_value_that_is_not_finite_stays_behind_the_diagonal(T, d, at, value):
    """A value row that is infinite or NaN reaches the queries that see it and no other, those that
    share its tile with a weight of zero among them."""
    O, LSE, (Oref, Lref) = run(1, 2, 1, T, d, 2, 90 + T, spoil=(at, value))
    assert np.abs(LSE - Lref).max() <= TOL
    if at:
        assert np.abs(O[:, :, :at] - Oref[:, :, :at]).max() <= TOL
    assert not np.isfinite(O[:, :, at:]).any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("depth", [False, True])
@pytest.mark.parametrize("T", [5, 40])
def test_f32_weights_below_the_smallest_normal_number(T, d, depth):
    """A key or a slot of weight e^-90 = 2^-129.8 and value 2^127 adds e^-90 2^127 / n = 0.14 / n to the
    output of the n other keys' zeros.  (The weight has 20 bits left: 1e-6 of the result.)"""
    z = torch.zeros(1, 2, T, d, device="cuda")
    Q, K, V = z.clone(), z.clone(), z.clone()
    Q[..., 0] = 1.0
    Kd = Vd = None
    if depth:
        Kd, Vd = (torch.zeros(1, 2, T, 8, d, device="cuda") for _ in range(2))
        Kd[:, :, :, 6, 0], Vd[:, :, :, 6] = -90.0, 2.0 ** 127
    else:
        K[:, :, 3, 0], V[:, :, 3] = -90.0, 2.0 ** 127
    O, _ = moda_attn_fwd(Q, K, V, Kd, Vd, scale=1.0)
    torch.cuda.synchronize()
    t = np.arange(T)
    n = t + 1 + 7 if depth else t.astype(float)
    want = np.where(depth | (t >= 3), np.exp(-90.0) * 2.0 ** 127 / np.maximum(n, 1), 0.0)
    assert np.abs(synth.to_f64(O) - want[None, None, :, None]).max() <= 2e-6


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(300, 16, 4, 1, 64, 3, None), (9, 64, 8, 8, 128, 2, 4), (9, 64, 8, 9, 64, 2, None),
                                              (1, 4, 2, 6, 64, 70, 72), (2, 8, 8, 7, 128, 70, None), (3, 3, 1, 5, 128, 0, None),
                                              (1, 2, 2, 2, 64, 0, 1)])
def test_f32_short_sequences(B, Hq, Hk, T, d, L, La, causal):
    """Both sides of the lines up to which a sequence's queries take a wave each; slots in one and in two steps
    of 64."""
    O, LSE, (Oref, Lref) = run(B, Hq, Hk, T, d, L, 300 + T + L, causal, La)
    assert np.abs(O - Oref).max() <= TOL and np.abs(LSE - Lref).max() <= TOL


@pytest.mark.parametrize("T,d,L,dead", [(4, 64, 3, 3), (6, 128, 70, 65), (200, 64, 12, 7)])
def test_f32_depth_slots_of_weight_zero(T, d, L, dead):
    """Slots whose scores are -inf weigh nothing, also where they are a row's first 64 or its only ones."""
    inp = synth.make_inputs(1, 2, 2, T, d, L, dtype="f32", seed=500, device="cuda")
    Q = inp["Q"].abs() + 0.1  # (positive: -inf, not NaN)
    inp["Kdepth"][:, :, :, :dead] = -float("inf")
    rest = [inp[k][:, :, :, dead:].contiguous() for k in ("Kdepth", "Vdepth")] if dead < L else [None, None]
    O, LSE = moda_attn_fwd(Q, inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"])
    O1, LSE1 = moda_attn_fwd(Q, inp["Kseq"], inp["Vseq"], *rest)
    torch.cuda.synchronize()
    assert (O - O1).abs().max().item() <= TOL and (LSE - LSE1).abs().max().item() <= TOL


@pytest.mark.parametrize("T,d,causal", [(100, 64, True), (70, 128, False), (161, 128, True)])
def test_f32_factors_without_three_parts(T, d, causal):
    """Factors that are not the sum of three finite bf16 numbers of normal size, in some tiles: keys of score
    -inf, a channel of values of 2^-120, a value that rounds to an infinite bf16.  (Channels are independent:
    1e-5 of each channel's largest value; scores, hence LSE, as everywhere.)"""
    inp = synth.make_inputs(1, 2, 1, T, d, 3, dtype="f32", seed=600 + T, device="cuda")
    inp["Q"][..., 0] = inp["Q"][..., 0].abs() + 0.1
    inp["Kseq"][:, :, 33:40, 0] = -float("inf")
    inp["Vseq"][..., 5] *= 2.0 ** -120
    inp["Vdepth"][..., 5] *= 2.0 ** -120
    inp["Vseq"][:, :, 20, 7] = 3.4e38
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"], causal=causal)
    torch.cuda.synchronize()
    Oref, Lref = R.fwd(*(synth.to_f64(inp[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), causal=causal)
    assert np.abs(synth.to_f64(LSE) - Lref).max() <= TOL
    scale = np.abs(Oref).max(axis=(0, 1, 2))
    assert (np.abs(synth.to_f64(O) - Oref).max(axis=(0, 1, 2)) <= TOL * scale.clip(min=2.0 ** -125)).all()


@pytest.mark.parametrize("T,d", [(300, 64), (200, 128)])
def test_f32_wide_scores(T, d):
    """Softmax scale 1: weights down to 2^-200.  An error of a score is an error of its weight: (d + 6) roundings
    of 2^-24 of sum |q k|, on both sides of the quotient."""
    inp = synth.make_inputs(1, 2, 2, T, d, 2, dtype="f32", seed=650 + T, device="cuda")
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"], scale=1.0)
    torch.cuda.synchronize()
    q, k, kd = (np.abs(synth.to_f64(inp[n])) for n in ("Q", "Kseq", "Kdepth"))
    size = max((q @ k.transpose(0, 1, 3, 2)).max(), (kd * q[:, :, :, None]).sum(-1).max())
    delta = (d + 6) * 2.0 ** -24 * size
    Oref, Lref = R.fwd(*(synth.to_f64(inp[n]) for n in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), scale=1.0)
    assert np.abs(synth.to_f64(O) - Oref).max() <= 2 * delta * float(max(inp["Vseq"].abs().max(), inp["Vdepth"].abs().max()))
    assert np.abs(synth.to_f64(LSE) - Lref).max() <= delta + TOL


@pytest.mark.parametrize("which,exponent", [("Q", -120), ("K", -120), ("Q", -112), ("K", -112)])
@pytest.mark.parametrize("T,d,causal", [(100, 64, True), (70, 128, False), (161, 128, True)])
def test_f32_minute_queries_or_keys(T, d, causal, which, exponent):
    """Queries of 2^-120 on keys of 2^120, and the other way round, for the heads of the first group: the last parts
    of such factors are below the range of bf16, their scores are of size 1."""
    inp = synth.make_inputs(1, 4, 2, T, d, 3, dtype="f32", seed=670 + T, device="cuda")
    f = 2.0 ** (exponent if which == "Q" else -exponent)
    inp["Q"][:, :2] *= f
    inp["Kseq"][:, :1] /= f
    inp["Kdepth"][:, :1] /= f
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"], causal=causal)
    torch.cuda.synchronize()
    Oref, Lref = R.fwd(*(synth.to_f64(inp[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), causal=causal)
    assert np.abs(synth.to_f64(O) - Oref).max() <= TOL and np.abs(synth.to_f64(LSE) - Lref).max() <= TOL


@pytest.mark.parametrize("T,d", [(100, 64), (161, 128)])
@pytest.mark.parametrize("causal", [True, False])
def test_f32_minute_values_beside_others(T, d, causal):
    """Values of 2^-120 with values of 1 in the same tile and channel, which the queries do not see (causal: rows
    before them) or give no weight (e^-300): 1e-5 of each channel's largest output."""
    inp = synth.make_inputs(1, 2, 1, T, d, 0, dtype="f32", seed=690 + T, device="cuda")
    inp["Vseq"] *= 2.0 ** -120
    for k0 in range(0, T, 32):
        inp["Vseq"][:, :, k0 + 16:k0 + 24] = 1.0
    rows = T
    if causal:
        rows = 16
    else:
        inp["Q"][..., 0] = 1.0
        inp["Kseq"][..., 0] = 0.0
        for k0 in range(0, T, 32):
            inp["Kseq"][:, :, k0 + 16:k0 + 24, 0] = -300.0 * d ** 0.5
    O, _ = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], causal=causal)
    torch.cuda.synchronize()
    Oref = R.fwd(*(synth.to_f64(inp[k]) for k in ("Q", "Kseq", "Vseq")), None, None, causal=causal)[0][:, :, :rows]
    scale = np.abs(Oref).max(axis=(0, 1, 2))
    assert scale.max() < 2.0 ** -110  # (the values of 1 take no part)
    assert (np.abs(synth.to_f64(O)[:, :, :rows] - Oref).max(axis=(0, 1, 2)) <= TOL * scale).all()


@pytest.mark.parametrize("d", [64, 128])
def test_f32_values_at_the_end_of_the_range(d):
    """253.6 * 2^120 with weights 1 and 0.0088: their sum is 255.8 * 2^120, below 2^128; that of the values rounded to
    bf16, 254 * 2^120, is not."""
    T, w, v = 40, 0.0088, 253.6 * 2.0 ** 120
    z = torch.zeros(1, 2, T, d, device="cuda")
    Q, K, V = z.clone(), z.clone(), z.clone()
    Q[..., 0] = 1.0
    K[..., 0] = -20.0  # (weights of 2e-9 on values of zero)
    K[:, :, 0, 0], K[:, :, 1, 0] = 0.0, float(np.log(w))
    V[:, :, :2] = v
    O, _ = moda_attn_fwd(Q, K, V, causal=False, scale=1.0)
    torch.cuda.synchronize()
    assert (np.abs(synth.to_f64(O) - v) <= 4 * 2.0 ** -24 * v).all()
