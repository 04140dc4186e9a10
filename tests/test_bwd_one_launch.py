"""GPU parity of the backward's one kernel for dK, dV and dQ: every kind of its tiles (key tiles of 128 or 32
keys, query tiles of 128 rows or 32 positions, four and eight waves) with 0, 1, 2 and 4 heads of depth slots, at
lengths on both sides of the tiles' edges.  Bound and oracle as in test_bwd_parity."""
import ctypes

import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import moda_attn_bwd, moda_attn_fwd, synth
from paper_2603_15619_amd.binding import MODAShape, lib
from test_bwd_parity import NAMES, compare, run_gpu

pytestmark = pytest.mark.gpu


def check(B, Hq, Hk, T, d, L, La, causal):
    """The first and the last sequence against the oracle; slots that are not attended hold NaN."""
    La = L if La is None else La
    s = MODAShape(B, Hq, Hk, T, d, La, L, int(causal), 0.0, 1)
    assert lib().moda_kernels_per_call(ctypes.byref(s), 1) == 2
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=2000 + T + L + d, device="cuda", depth_alloc=La, with_dO=True)
    if La > L:
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    grads = run_gpu(inp, L, causal)
    for b in {0, B - 1}:
        one = {k: None if v is None else v[b:b + 1].clone() for k, v in inp.items()}
        if La > L:
            one["Kdepth"][:, :, :, L:] = 0
            one["Vdepth"][:, :, :, L:] = 0
        args = [None if one[k] is None else synth.to_f64(one[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth", "dO")]
        ref, noise = R.bwd(*args, depth_count=L, causal=causal), R.bwd_noise(*args, depth_count=L, causal=causal)
        for name, g, r, n in zip(NAMES, grads, ref, noise):
            if g is not None:
                compare(name, g[b:b + 1], r, n)
    for g in grads:
        assert g is None or torch.isfinite(g.float()).all()
    if La > L:
        assert torch.count_nonzero(grads[3][:, :, :, L:].float()) == 0 and torch.count_nonzero(grads[4][:, :, :, L:].float()) == 0


EIGHT_128 = [(2, 1, 1, 127, 12, 13, True), (1, 1, 1, 17, 12, None, False), (2, 2, 1, 97, 12, None, True), (1, 2, 1, 500, 3, 4, False), (4, 4, 1, 200, 1, None, True),
             (1, 4, 1, 33, 1, 2, False), (3, 1, 1, 257, 0, None, True), (2, 3, 1, 161, 0, None, False), (8, 8, 1, 33, 0, None, True),
             (16, 8, 1, 127, 0, None, True), (8, 8, 1, 257, 0, None, False), (2, 32, 4, 300, 0, None, True)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hk,T,L,La", [(1, 1, 1, 17, 3, 4), (2, 3, 3, 33, 6, None), (1, 2, 2, 127, 5, 9), (1, 4, 2, 31, 4, None),
                                            (3, 2, 1, 65, 12, 13), (1, 4, 1, 32, 7, 8), (2, 8, 2, 97, 2, None), (1, 6, 6, 129, 0, 3),
                                            (1, 1, 1, 161, 0, None), (2, 3, 1, 63, 0, None), (1, 5, 1, 17, 0, None),
                                            (16, 2, 1, 33, 3, 4), (40, 4, 1, 33, 5, None)])
def test_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    """32 keys and 32 positions to a workgroup (d = 128: of four waves, or eight where groups or slots are longest)."""
    check(B, Hq, Hk, T, d, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(24, 3, 3, 97, 64, 1, 3, False), (30, 4, 4, 129, 128, 3, None, True), (72, 2, 1, 97, 64, 4, 5, False),
                                                     (40, 2, 1, 300, 128, 12, None, True), (200, 4, 1, 97, 128, 3, None, False), (15, 10, 5, 333, 64, 5, 6, True),
                                                     (33, 4, 1, 500, 64, 3, None, True), (40, 3, 3, 257, 64, 0, None, True), (40, 3, 3, 257, 128, 0, None, False),
                                                     (72, 8, 1, 500, 64, 0, None, True), (41, 1, 1, 700, 128, 15, 16, True), (83, 1, 1, 530, 64, 12, None, False)])
def test_many_tiles(B, Hq, Hk, T, d, L, La, causal):
    """128 keys and 128 rows to a workgroup, heads that the dies divide evenly and others, walked tile by tile or with
    the key tiles spread among the query tiles (the last two, and 15 sequences of five heads)."""
    check(B, Hq, Hk, T, d, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(16, 16, 4, 500, 64, 0, None, True), (16, 8, 4, 900, 128, 1, 2, False), (24, 4, 1, 1500, 64, 3, None, True)])
def test_heads_of_a_die_together(B, Hq, Hk, T, d, L, La, causal):
    """More than 1024 workgroups with up to 1024 key tiles that are most of the work: a die walks all its heads at once."""
    check(B, Hq, Hk, T, d, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(16, 4, 1, 500, 128, 5, 6, True), (16, 4, 1, 97, 128, 1, None, False), (4, 2, 1, 1100, 128, 1, None, False),
                                                     (24, 2, 1, 300, 128, 1, 2, False), (16, 4, 1, 97, 64, 3, None, False), (8, 4, 1, 1000, 64, 5, None, True),
                                                     (40, 1, 1, 257, 128, 0, None, True), (9, 3, 1, 300, 128, 0, None, False), (24, 8, 1, 129, 128, 0, None, True),
                                                     (33, 8, 1, 127, 64, 0, None, False), (16, 3, 1, 500, 64, 0, None, True)])
def test_few_key_tiles_of_many_rows(B, Hq, Hk, T, d, L, La, causal):
    """32 keys and 128 rows to a workgroup."""
    check(B, Hq, Hk, T, d, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", [(1, 1, 1, 700, 5, 6, True), (1, 1, 1, 257, 1, None, False), (3, 2, 1, 200, 5, None, True), (1, 2, 1, 129, 13, 14, False),
                                                   (3, 4, 1, 300, 1, 2, True), (1, 4, 1, 65, 9, None, False), (1, 3, 1, 257, 0, None, True), (2, 8, 1, 97, 0, None, False),
                                                   (9, 8, 1, 129, 0, None, True), (2, 32, 2, 33, 0, None, True), (9, 8, 1, 127, 0, None, False)])
def test_eight_waves(B, Hq, Hk, T, L, La, causal):
    """d = 64: eight waves to a workgroup, 32 positions or (the last ones) 256 rows of dQ."""
    check(B, Hq, Hk, T, 64, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", EIGHT_128)
def test_eight_waves_d_128(B, Hq, Hk, T, L, La, causal):
    """... and at d = 128."""
    check(B, Hq, Hk, T, 128, L, La, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,d", [(11, 8, 1, 430, 64), (1, 64, 8, 399, 64), (9, 16, 1, 498, 128), (1, 32, 4, 1311, 128)])
def test_eight_waves_and_128_rows_in_one_to_two_rounds(B, Hq, Hk, T, d):
    """257 to 512 causal workgroups, of which a unit holds one at a time: the walk is not folded over two layers."""
    check(B, Hq, Hk, T, d, 0, None, True)


@pytest.mark.parametrize("Hq,T", [(2, 97), (4, 97), (8, 97)])
def test_slots_that_are_not_finite_reach_their_own_position_only(Hq, T):
    """(O and LSE are those of finite slots: the forward of several heads per tile makes no such promise.)"""
    G = Hq // 2
    inp = synth.make_inputs(1, Hq, Hq // G, T, 128, 6, dtype="bf16", seed=77, device="cuda", with_dO=True)
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"])

    def grads():
        return moda_attn_bwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"], O, LSE, inp["dO"])

    clean = grads()
    inp["Vdepth"][0, 1, 50, 5, 3] = float("inf")
    got = grads()
    keep = torch.ones(T, dtype=torch.bool, device="cuda")
    keep[50] = False
    for i in (1, 2):
        assert torch.equal(got[i], clean[i])
    for i in (0, 3, 4):
        assert torch.equal(got[i][:, :, keep], clean[i][:, :, keep])
    assert torch.equal(got[0][:, :G], clean[0][:, :G]) and not torch.isfinite(got[0][0, G, 50].float()).all()
