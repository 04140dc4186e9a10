"""GPU parity: bf16 forward kernel (through the C ABI) where the reference of the exponentials, which the
key loop takes from the tiles before, is far too low for a tile: scores that jump by hundreds of
powers of two at single keys (weights formed with the old reference overflow to infinity), in every ring
stage, in the first, the last and the remaining tiles of a wave; and first tiles, or first depth slots, whose
scores are all -inf.  The oracle is the fp64 forward in C.

Tolerance: one key carries a row, so |O| reaches max|V|: weights and output rounded to bf16, 2 * 2^-8 *
max|V|.  LSE (up to 1000 in size): 1e-3 as in test_fwd_parity plus four fp32 roundings of its size.
"""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import synth

from test_fwd_parity import run_gpu

pytestmark = pytest.mark.gpu


def check(inp, B, Hq, Hk, T, d, L, causal, tuning, first_row=0):
    print("case", dict(Hq=Hq, Hk=Hk, T=T, d=d, L=L, causal=causal, tuning=tuning), flush=True)
    O, LSE = run_gpu(inp, L, causal, None, tuning)
    with np.errstate(invalid="ignore"):
        Oref, Lref = R.fwd(*(synth.to_f64(inp[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")),
                           depth_count=L, causal=causal)
    vmax = max(float(inp[k].abs().max()) for k in (("Vseq", "Vdepth") if L else ("Vseq",)))
    o, l = synth.to_f64(O)[:, :, first_row:], synth.to_f64(LSE)[:, :, first_row:]
    Oref, Lref = Oref[:, :, first_row:], Lref[:, :, first_row:]
    assert np.isfinite(o).all() and np.isfinite(l).all()
    assert np.abs(o - Oref).max() <= 2 * 2.0 ** -8 * vmax
    assert (np.abs(l - Lref) <= 1e-3 + 4 * 2.0 ** -24 * np.abs(Lref)).all()


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("Hk,T,d,L,causal", [(4, 580, 64, 0, True), (4, 711, 128, 3, True), (2, 650, 64, 6, True),
                                             (2, 523, 128, 0, False), (4, 390, 64, 5, False), (1, 777, 128, 2, True)])
def test_scores_that_jump(waves, Hk, T, d, L, causal):
    B, Hq = 2, 4
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=900 + T, device="cuda")
    for pos, factor in ((0, 8.0), (40, 30.0), (63, 60.0), (70, 200.0), (130, 250.0), (200, 300.0), (290, 350.0),
                        (350, 20.0), (T - 1, 400.0)):
        inp["Kseq"][:, :, pos] *= factor
    check(inp, B, Hq, Hk, T, d, L, causal, dict(waves=waves))


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("T,d,L", [(300, 64, 0), (450, 128, 0), (330, 128, 4)])
def test_first_tiles_of_minus_infinity(waves, T, d, L):
    """70 keys (the first tile and a few more) of score -inf: rows that see others are as if those keys were not
    there.  (Without depth slots the first rows see nothing else: their softmax is not defined.)"""
    B, Hq, Hk, blocked = 2, 2, 2, 70
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=950 + T, device="cuda")
    inp["Q"][..., 0] = inp["Q"][..., 0].abs() + 0.25
    inp["Kseq"][:, :, :blocked, 0] = -float("inf")
    check(inp, B, Hq, Hk, T, d, L, True, dict(waves=waves), first_row=0 if L else blocked)


# Both geometries of both head dimensions, at d = 64 two and four waves per SIMD (few and many workgroups);
# workgroups that take their slots before the key loop and after it.
KERNELS = [(2, 4, 300, 64, 4), (50, 4, 300, 64, 4), (50, 4, 300, 64, 8), (2, 4, 300, 128, 4), (2, 4, 300, 128, 8)]


@pytest.mark.parametrize("offset", [-2048.0, 2048.0])
@pytest.mark.parametrize("Hk,L", [(4, 0), (4, 5), (2, 5)])
@pytest.mark.parametrize("B,H,T,d,waves", KERNELS)
def test_far_scores_behind_first_tiles_of_minus_infinity(B, H, T, d, waves, Hk, L, offset):
    """70 keys of score -inf, all other keys and slots `offset` away from zero (+-261 and +-369 powers of two):
    the softmax is that without the offset, whatever reference the empty first tiles left."""
    inp = synth.make_inputs(B, H, Hk, T, d, L, dtype="bf16", seed=970 + L, device="cuda")
    blocked = 70
    inp["Q"][..., 0] = inp["Q"][..., 0].abs() + 0.25
    inp["Q"][..., 1] = 32.0
    inp["Kseq"][..., 1] = offset / 32.0
    inp["Kseq"][:, :, :blocked, 0] = -float("inf")
    if L:
        inp["Kdepth"][..., 1] = offset / 32.0
    O, LSE = run_gpu(inp, L, True, None, dict(waves=waves))
    for b in (0, B - 1):
        one = {k: None if v is None else v[b:b + 1].contiguous() for k, v in inp.items()}
        with np.errstate(invalid="ignore"):
            Oref, Lref = R.fwd(*(synth.to_f64(one[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), depth_count=L)
        rows = slice(0 if L else blocked, T)
        o, l, Oref, Lref = (x[:, :, rows] for x in (synth.to_f64(O[b:b + 1]), synth.to_f64(LSE[b:b + 1]), Oref, Lref))
        vmax = max(float(one[k].abs().max()) for k in (("Vseq", "Vdepth") if L else ("Vseq",)))
        # (weights are formed from scores of size 2048 in fp32: 2^-13 of each, next to their rounding to bf16)
        assert np.abs(o - Oref).max() <= 2 * 2.0 ** -8 * vmax
        assert (np.abs(l - Lref) <= 1e-3 + 4 * 2.0 ** -24 * np.abs(Lref)).all()


@pytest.mark.parametrize("L,dead", [(12, 12), (7, 3), (12, 5), (12, 10)])
@pytest.mark.parametrize("B,H,T,d,waves", KERNELS)
def test_depth_slots_of_weight_zero(B, H, T, d, waves, L, dead):
    """One head per tile: slots whose scores are -inf, all of a row's or one or two whole work items (of 3 or 5
    slots) among them, weigh nothing: the result is that without them (the other slots' weights round to
    bf16 as before: 2e-2 on O)."""
    inp = synth.make_inputs(B, H, H, T, d, L, dtype="bf16", seed=960 + L, device="cuda")
    inp["Q"] = inp["Q"].abs() + 0.1  # (positive: -inf, not NaN)
    rest = dict(inp, Kdepth=inp["Kdepth"][:, :, :, dead:].contiguous(), Vdepth=inp["Vdepth"][:, :, :, dead:].contiguous())
    if dead == L:
        rest["Kdepth"] = rest["Vdepth"] = None
    O1, L1 = run_gpu(rest, L - dead, tuning=dict(waves=waves))
    inp["Kdepth"][:, :, :, :dead] = -float("inf")
    O, LSE = run_gpu(inp, L, tuning=dict(waves=waves))
    assert (O.float() - O1.float()).abs().max().item() <= 2e-2
    assert (LSE - L1).abs().max().item() <= 1e-4


@pytest.mark.parametrize("T,d", [(1000, 128), (1500, 64)])
def test_rows_that_one_key_carries(T, d):
    """A grid of one round, whose light tiles take their slots first: a key 6 to 7.5 powers of two above them weighs
    exactly 1, whatever the slots' reference: |O| is off by its own rounding (2^-8) and that of the slots' weights
    (2^-8 of the seven slots' share, 7 * 2^-6)."""
    B, H, L = 2, 16, 7
    inp = synth.make_inputs(B, H, H, T, d, L, dtype="bf16", seed=990, device="cuda")
    jitter = 1.0 + 0.25 * torch.rand(B, H, T, device="cuda")
    for k in ("Q", "Kseq", "Kdepth"):
        inp[k].zero_()
    inp["Q"][..., 0] = jitter.to(torch.bfloat16)
    inp["Kseq"][:, :, :, 0] = -40.0
    inp["Kseq"][:, :, 0, 0] = 6.0
    inp["Vseq"][:, :, 0] = inp["Vseq"][:, :, 0].abs() + 1.0
    inp["Vdepth"] = inp["Vdepth"].clamp(-1.0, 1.0)
    scale = float(np.log(2.0))
    O, _ = run_gpu(inp, L, True, scale)
    Oref, _ = R.fwd(*(synth.to_f64(inp[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), depth_count=L, scale=scale)
    assert (np.abs(synth.to_f64(O) - Oref) <= 2.0 ** -8 * (np.abs(Oref) + 7 * 2.0 ** -6) + 1e-5).all()


@pytest.mark.parametrize("L", [0, 3])
@pytest.mark.parametrize("B,H,T,d,waves", KERNELS)
def test_raised_reference_is_the_largest_score(B, H, T, d, waves, L):
    """Key 100 is 12 to 13.5 powers of two above the keys before it, key 250 another 28 to 31.5: it weighs exactly 1 and all
    others, together below 300 * 2^-28, nothing, so that the rows behind it are its value, bit by bit."""
    inp = synth.make_inputs(B, H, H, T, d, L, dtype="bf16", seed=1000 + d, device="cuda")
    for k in ("Q", "Kseq", "Kdepth"):
        if inp[k] is not None:
            inp[k].zero_()
    inp["Q"][..., 0] = (1.0 + 0.125 * torch.rand(B, H, T, device="cuda")).to(torch.bfloat16)
    inp["Kseq"][:, :, 100, 0], inp["Kseq"][:, :, 250, 0] = 12.0, 40.0
    inp["Vseq"] = inp["Vseq"].sign() * (inp["Vseq"].abs() + 2.0 ** -6)  # (no value so small that the others' share shows)
    O, LSE = run_gpu(inp, L, True, float(np.log(2.0)), dict(waves=waves))
    assert torch.equal(O[:, :, 250:], inp["Vseq"][:, :, 250:251].expand(-1, -1, T - 250, -1))
    assert (LSE[:, :, 250:] / float(np.log(2.0)) - 40.0 * inp["Q"][:, :, 250:, 0].float()).abs().max().item() <= 1e-4


@pytest.mark.parametrize("B,H,T,d,waves", [(B, H, 250, d, waves) for B, H, _, d, waves in KERNELS])
def test_references_leave_out_masked_keys(B, H, T, d, waves):
    """Every key is 32 powers of two above the one before it: a row's last key carries it, and the keys that it does not
    see, up to 8000 powers above, must not become its reference."""
    inp = synth.make_inputs(B, H, H, T, d, 0, dtype="bf16", seed=1010 + d, device="cuda")
    inp["Q"].zero_()
    inp["Kseq"].zero_()
    inp["Q"][..., 0] = 32.0
    inp["Kseq"][..., 0] = torch.arange(T, device="cuda").to(torch.bfloat16)
    inp["Vseq"] = inp["Vseq"].sign() * (inp["Vseq"].abs() + 2.0 ** -6)
    O, LSE = run_gpu(inp, 0, True, float(np.log(2.0)), dict(waves=waves))
    assert torch.equal(O, inp["Vseq"])
    want = torch.arange(T, device="cuda").float() * float(32 * np.log(2.0))
    assert ((LSE - want).abs() <= 4 * 2.0 ** -24 * want + 1e-6).all()
