"""GPU parity of the bf16 forward for calls with few tiles (32 (position, head) pairs per workgroup,
key tiles and blocks of depth slots dealt out to its waves), and of the rule that picks it: both
kernels on the same inputs.  Tolerances as in test_fwd_parity."""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import synth
from test_fwd_parity import check_full, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 2, 3), (1, 2, 2, 31, 128, 5, None), (2, 2, 2, 32, 64, 6, 8),
                                              (1, 3, 3, 33, 128, 11, None), (1, 2, 2, 129, 64, 31, None), (2, 4, 2, 63, 128, 3, 4),
                                              (1, 8, 1, 97, 64, 9, 10), (1, 32, 1, 65, 128, 1, None), (1, 64, 1, 40, 64, 33, 34), (3, 32, 8, 200, 64, 5, None),
                                              (1, 12, 2, 161, 128, 0, 2), (1, 4, 1, 1030, 64, 7, None)])
def test_fwd_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=1500 + T + L, device="cuda", depth_alloc=La)
    if La is not None:  # unattended slots take no part
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    check_full(B, Hq, Hk, T, d, L, "bf16", 0, causal=causal, depth_alloc=La, inp=inp)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(2, 16, 8, 1000, 64, 12, 13, True), (5, 8, 4, 485, 64, 24, None, False), (3, 32, 8, 226, 64, 31, 32, True),
                                                     (1, 64, 8, 300, 64, 64, None, True), (1, 16, 8, 1100, 128, 12, None, True), (1, 16, 4, 1069, 128, 24, 25, True)])
def test_blocks_of_slots_first_in_every_other_workgroup(B, Hq, Hk, T, d, L, La, causal):
    """Two, four and eight heads per tile, more workgroups than two per unit, five slots and more to a head of the
    group; the slots of the first position score -inf
    (its query is positive), so that a workgroup's first block holds columns that have seen no key yet."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=1550 + T + L, device="cuda", depth_alloc=La)
    inp["Q"][:, :, 0] = inp["Q"][:, :, 0].abs() + 0.1
    inp["Kdepth"][:, :, 0] = -float("inf")
    inp["Vdepth"][:, :, 0] = 0.0  # (weight zero either way)
    if La is not None:
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    O, LSE = run_gpu(inp, L, causal)
    finite = dict(inp, Kdepth=inp["Kdepth"].clone())
    finite["Kdepth"][:, :, 0] = torch.where(torch.isneginf(finite["Kdepth"][:, :, 0]), -1e4, finite["Kdepth"][:, :, 0])  # (scores below -1e3: weight zero)
    args = [synth.to_f64(finite[k][:1]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")]
    Oref, Lref = R.fwd(*(np.nan_to_num(a) for a in args), depth_count=L, causal=causal)
    assert np.abs(synth.to_f64(O[:1]) - Oref).max() <= 2e-2 and np.abs(synth.to_f64(LSE[:1]) - Lref).max() <= 1e-3
    assert torch.isfinite(O.float()).all() and torch.isfinite(LSE).all()


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,causal", [(1, 8, 8, 700, 64, 4, True), (1, 8, 2, 513, 128, 6, True),
                                                  (1, 16, 2, 300, 64, 0, False), (1, 2, 2, 4100, 128, 1, True),
                                                  (1, 12, 12, 4096, 64, 0, True), (1, 3, 3, 9000, 128, 2, True), (1, 12, 12, 2000, 64, 0, False),
                                                  (1, 4, 4, 3900, 128, 0, False)])
def test_both_kernels_agree(B, Hq, Hk, T, d, L, causal):
    """(an empty tuning keeps the other kernel).  Both round weights and outputs to bf16: 2e-2 on O."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=1600 + T, device="cuda")
    O0, L0 = run_gpu(inp, L, causal)
    O1, L1 = run_gpu(inp, L, causal, tuning={})
    assert (O0.float() - O1.float()).abs().max().item() <= 2e-2
    assert (L0 - L1).abs().max().item() <= 1e-4


@pytest.mark.parametrize("T,d,at", [(70, 64, 37), (200, 128, 130)])
def test_depth_values_that_are_not_finite_stay_in_their_row(T, d, at):
    """One head per tile: an infinite value in a depth slot reaches its own position only."""
    inp = synth.make_inputs(1, 2, 2, T, d, 3, dtype="bf16", seed=1700, device="cuda")
    clean, _ = run_gpu(inp, 3)
    inp["Vdepth"][:, :, at, 1] = float("inf")
    O, _ = run_gpu(inp, 3)
    keep = [t for t in range(T) if t != at]
    assert torch.equal(O[:, :, keep], clean[:, :, keep])
    assert not torch.isfinite(O[:, :, at].float()).any()


@pytest.mark.parametrize("T,d,L,dead", [(200, 64, 6, 6), (130, 128, 12, 12), (200, 64, 12, 7), (97, 128, 5, 5)])
def test_depth_slots_of_weight_zero(T, d, L, dead):
    """One head per tile: slots whose scores are -inf, all of a row's or a whole step's among them, weigh
    nothing: the result is that without them (the other slots' weights round to bf16 as before: 2e-2 on O)."""
    inp = synth.make_inputs(1, 2, 2, T, d, L, dtype="bf16", seed=1800, device="cuda")
    inp["Q"] = inp["Q"].abs() + 0.1  # (positive: -inf, not NaN)
    rest = dict(inp, Kdepth=inp["Kdepth"][:, :, :, dead:].contiguous(), Vdepth=inp["Vdepth"][:, :, :, dead:].contiguous())
    if dead == L:
        rest["Kdepth"] = rest["Vdepth"] = None
    O1, L1 = run_gpu(rest, L - dead)
    inp["Kdepth"][:, :, :, :dead] = -float("inf")
    O, LSE = run_gpu(inp, L)
    assert (O.float() - O1.float()).abs().max().item() <= 2e-2
    assert (LSE - L1).abs().max().item() <= 1e-4


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,causal", [(64, 16, 16, 100, 64, 3, True), (40, 8, 8, 384, 128, 0, False),
                                                  (40, 16, 4, 128, 64, 5, True), (12, 16, 16, 500, 64, 2, True),
                                                  (6, 8, 8, 1800, 128, 0, False), (8, 16, 16, 513, 128, 1, True),
                                                  (7, 12, 12, 1030, 128, 1, True), (29, 4, 4, 1000, 128, 0, True),
                                                  (13, 12, 12, 1030, 64, 2, True)])
def test_workgroups_of_four_waves(B, Hq, Hk, T, d, L, causal):
    """Short sequences in large grids and one and a half rounds of workgroups take four waves (the last three
    cases just do not, see test_abi's kernel names): against eight on the same inputs, rows of whole heads
    against the oracle."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=1900 + T, device="cuda")
    O0, L0 = run_gpu(inp, L, causal)
    O1, L1 = run_gpu(inp, L, causal, tuning=dict(waves=8))
    assert (O0.float() - O1.float()).abs().max().item() <= 2e-2
    assert (L0 - L1).abs().max().item() <= 1e-4
    one = {k: None if v is None else v[B - 1:].contiguous() for k, v in inp.items()}
    Oref, Lref = R.fwd(*(synth.to_f64(one[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), depth_count=L, causal=causal)
    assert np.abs(synth.to_f64(O0[B - 1:]) - Oref).max() <= 2e-2
    assert np.abs(synth.to_f64(L0[B - 1:]) - Lref).max() <= 1e-3


@pytest.mark.parametrize("B,Hq,Hk,T,L,causal", [(3, 11, 11, 1300, 2, True), (5, 13, 13, 700, 0, True), (3, 10, 5, 1290, 3, True),
                                                (2, 23, 23, 1100, 1, False)])
def test_grids_of_one_round(B, Hq, Hk, T, L, causal):
    """d = 128, more than 256 workgroups of four waves that are resident all at once (tiles of every other layer in
    reverse where causal; 8 does not divide their number), slots first in the light tiles."""
    check_ends(B, Hq, Hk, T, 128, L, 1950 + T, causal)


@pytest.mark.parametrize("d,B,H,T,L", [(128, 14, 14, 100, 7), (128, 14, 14, 100, 6), (64, 30, 14, 100, 14), (64, 30, 14, 128, 10),
                                       (128, 14, 17, 129, 7), (128, 16, 16, 250, 8), (128, 16, 14, 250, 8), (128, 40, 13, 240, 12),
                                       (128, 40, 13, 230, 12), (128, 40, 13, 500, 12), (128, 16, 16, 240, 13), (128, 16, 8, 490, 12)])
def test_heads_of_one_or_two_tiles(d, B, H, T, L):
    """Either side of the lines between slots first in the light half (in no tile, where a head has one) and in every
    other workgroup, and between four and eight waves for many slots."""
    check_ends(B, H, H, T, d, L, 1970 + T, True)


def check_ends(B, Hq, Hk, T, d, L, seed, causal):
    """The first and the last sequence (they differ in their data only)."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=seed, device="cuda")
    O, LSE = run_gpu(inp, L, causal)
    for b in (0, B - 1):
        one = {k: None if v is None else v[b:b + 1].contiguous() for k, v in inp.items()}
        Oref, Lref = R.fwd(*(synth.to_f64(one[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")), depth_count=L, causal=causal)
        assert np.abs(synth.to_f64(O[b:b + 1]) - Oref).max() <= 2e-2
        assert np.abs(synth.to_f64(LSE[b:b + 1]) - Lref).max() <= 1e-3
