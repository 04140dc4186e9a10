"""GPU parity of the backward's one kernel for dK, dV and dQ: every kind of its tiles (key tiles of 128 or 32
keys, query tiles of 128 rows or 32 positions, four and eight waves) with 0, 1, 2 and 4 heads of depth slots, at
lengths on both sides of the tiles' edges.  Bound and oracle as in test_bwd_parity."""
import ctypes
import math
import re

import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import moda_attn_bwd, moda_attn_fwd, synth
from paper_2603_15619_amd.binding import MODAShape, lib
from test_bwd_parity import NAMES, compare, run_gpu

pytestmark = pytest.mark.gpu


def route(B, Hq, Hk, T, d, L, La, causal):
    """(32 keys to a key tile, 32 positions to a query tile, waves), workgroups and key tiles of the call's one launch."""
    s = MODAShape(B, Hq, Hk, T, d, La, L, int(causal), 0.0, 1)
    assert lib().moda_kernels_per_call(ctypes.byref(s), 1) == 2
    name = ctypes.create_string_buffer(64)
    lib().moda_bwd_kernel_name(ctypes.byref(s), 1, name, len(name))
    m = re.match(r"moda_bwd_grads_kernel<(\d+), (\d), (\w+), (\w+), (\d)>", name.value.decode())
    G = Hq // Hk
    assert int(m[1]) == d and int(m[2]) == (0 if La == 0 else G)
    keys, queries, waves = m[3] == "true", m[4] == "true", int(m[5])
    heads = G if La > 0 else 1 if queries else math.gcd(G, 4)
    key_tiles = B * Hk * -(-T // (32 if keys else 128))
    return (keys, queries, waves), key_tiles + B * Hk * (G // heads) * -(-T // (32 if queries else waves * 32 // heads)), key_tiles


def check(B, Hq, Hk, T, d, L, La, causal, kind):
    """The first and the last sequence against the oracle; slots that are not attended hold NaN.  `kind`: as of route (4
    or 8 waves where it names none)."""
    La = L if La is None else La
    assert route(B, Hq, Hk, T, d, L, La, causal)[0][:len(kind)] == kind
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
             (1, 4, 1, 33, 4, 5, False), (5, 4, 1, 2100, 1, 2, False), (1, 2, 1, 257, 0, None, True), (2, 3, 1, 161, 0, None, False), (8, 8, 1, 33, 0, None, True),
             (16, 8, 1, 127, 0, None, True), (8, 8, 1, 257, 0, None, False), (2, 32, 4, 300, 0, None, True)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hk,T,L,La", [(1, 1, 1, 17, 3, 4), (2, 3, 3, 33, 6, None), (1, 2, 2, 127, 5, 9), (1, 4, 2, 31, 4, None),
                                            (3, 2, 1, 65, 12, 13), (1, 4, 1, 32, 7, 8), (2, 8, 2, 129, 2, None), (1, 6, 6, 129, 0, 3),
                                            (1, 1, 1, 161, 0, None), (2, 3, 1, 63, 0, None), (1, 5, 1, 17, 0, None),
                                            (16, 2, 1, 33, 3, 4), (40, 2, 1, 33, 5, None)])
def test_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    """32 keys and 32 positions to a workgroup of four waves, or eight where groups or slots are longest."""
    check(B, Hq, Hk, T, d, L, La, causal, (True, True))


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(33, 4, 4, 65, 64, 1, 3, False), (30, 4, 4, 129, 128, 3, None, True), (72, 2, 1, 161, 64, 1, 2, False),
                                                     (40, 2, 1, 300, 128, 12, None, True), (200, 4, 1, 97, 128, 3, None, False), (15, 10, 5, 333, 64, 5, 6, True),
                                                     (3, 32, 8, 253, 64, 64, None, True), (40, 3, 3, 257, 64, 0, None, True), (40, 3, 3, 257, 128, 0, None, False),
                                                     (72, 8, 1, 333, 64, 0, None, False), (41, 1, 1, 700, 128, 15, 16, True), (83, 1, 1, 530, 64, 12, None, False)])
def test_many_tiles(B, Hq, Hk, T, d, L, La, causal):
    """128 keys and 128 rows to a workgroup, heads that the dies divide evenly and others, walked tile by tile."""
    check(B, Hq, Hk, T, d, L, La, causal, (False, False, 4))


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal,kind", [(41, 1, 1, 2100, 128, 15, 16, True, (False, False, 4)), (83, 1, 1, 1000, 64, 12, None, False, (False, False, 4)),
                                                          (15, 10, 5, 700, 64, 5, 6, True, (False, False, 4)), (15, 20, 5, 500, 64, 5, None, True, (False, False, 4)),
                                                          (3, 4, 4, 1601, 128, 7, 8, True, (True, True, 4))])
def test_key_tiles_among_the_query_tiles(B, Hq, Hk, T, d, L, La, causal, kind):
    """Heads that 8 does not divide, more than two rounds of workgroups, slots as long as the key tiles: the key tiles are
    spread evenly among the query tiles."""
    grid = route(B, Hq, Hk, T, d, L, L if La is None else La, causal)[1]
    assert B * Hk % 8 != 0 and grid > 1024 and L >= 4 and T * (Hq // Hk) <= 600 * L
    check(B, Hq, Hk, T, d, L, La, causal, kind)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(16, 16, 4, 500, 64, 0, None, True), (16, 8, 4, 900, 128, 1, 2, False), (72, 8, 2, 161, 64, 1, None, False)])
def test_heads_of_a_die_together(B, Hq, Hk, T, d, L, La, causal):
    """More than 1024 workgroups with up to 1024 key tiles that are most of the work: a die walks all its heads at once."""
    kind, grid, key_tiles = route(B, Hq, Hk, T, d, L, L if La is None else La, causal)
    assert B * Hk % 8 == 0 and grid > 1024 >= key_tiles and T * (Hq // Hk) > 400 * L
    check(B, Hq, Hk, T, d, L, La, causal, kind)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(16, 4, 1, 500, 128, 5, 6, True), (16, 4, 1, 97, 128, 1, None, False), (24, 4, 2, 161, 128, 1, None, True),
                                                     (24, 2, 1, 300, 128, 1, 2, False), (16, 4, 1, 97, 64, 3, None, False), (3, 8, 2, 1001, 64, 5, None, False),
                                                     (9, 2, 1, 1001, 64, 1, 2, False), (8, 2, 2, 1001, 128, 1, None, False),
                                                     (40, 2, 1, 33, 128, 0, None, True), (9, 3, 1, 300, 128, 0, None, False), (24, 8, 1, 129, 128, 0, None, True),
                                                     (33, 8, 1, 127, 64, 0, None, False), (16, 3, 1, 500, 64, 0, None, True)])
def test_few_key_tiles_of_many_rows(B, Hq, Hk, T, d, L, La, causal):
    """32 keys and 128 rows to a workgroup."""
    check(B, Hq, Hk, T, d, L, La, causal, (True, False, 4))


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", [(1, 1, 1, 700, 5, 6, True), (1, 1, 1, 1001, 1, None, False), (3, 2, 1, 200, 5, None, True), (1, 2, 1, 129, 13, 14, False),
                                                   (3, 4, 1, 300, 1, 2, True), (1, 4, 1, 161, 9, None, False), (1, 3, 1, 257, 0, None, True), (2, 8, 1, 97, 0, None, False),
                                                   (9, 8, 1, 129, 0, None, True), (2, 32, 2, 33, 0, None, True), (9, 8, 1, 127, 0, None, False)])
def test_eight_waves(B, Hq, Hk, T, L, La, causal):
    """d = 64: eight waves to a workgroup, 32 positions or (the last ones) 256 rows of dQ."""
    assert route(B, Hq, Hk, T, 64, L, L if La is None else La, causal)[0][2] == 8
    check(B, Hq, Hk, T, 64, L, La, causal, (True,))


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", EIGHT_128)
def test_eight_waves_d_128(B, Hq, Hk, T, L, La, causal):
    """... and at d = 128."""
    assert route(B, Hq, Hk, T, 128, L, L if La is None else La, causal)[0][2] == 8
    check(B, Hq, Hk, T, 128, L, La, causal, (True,))


@pytest.mark.parametrize("B,Hq,Hk,T,d", [(11, 8, 1, 430, 64), (16, 8, 1, 257, 64), (9, 16, 1, 498, 128), (1, 32, 4, 1311, 128)])
def test_eight_waves_and_128_rows_in_one_to_two_rounds(B, Hq, Hk, T, d):
    """257 to 512 causal workgroups, of which a unit holds one at a time: the walk is not folded over two layers."""
    assert 256 < route(B, Hq, Hk, T, d, 0, 0, True)[1] <= 512
    check(B, Hq, Hk, T, d, 0, None, True, (True, False, 8))


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


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(16, 16, 2, 225, 64, 0), (24, 8, 1, 129, 128, 0), (40, 3, 3, 257, 128, 0), (30, 4, 4, 129, 128, 3), (200, 4, 1, 97, 128, 3),
                                           (24, 24, 8, 200, 64, 2), (24, 40, 8, 130, 128, 1), (1, 2, 2, 161, 64, 5)])
def test_key_that_is_not_finite_leaves_the_query_blocks_before_it_alone(B, Hq, Hk, T, d, L):
    """Causal: an infinite value, or a NaN key, at position j reaches dQ of the queries that see it and, as a product with weight
    zero, at most of those from the last multiple of 32 on (all kinds of query tiles, in one launch or of their own)."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=79, device="cuda", with_dO=True)
    args = [inp[k] for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")]
    O, LSE = moda_attn_fwd(*args)
    clean = moda_attn_bwd(*args, O, LSE, inp["dO"])[0].clone()
    j = T // 2 // 32 * 32 + 5
    for k, v in (("Vseq", float("inf")), ("Kseq", float("nan"))):
        old = inp[k][-1, -1, j, 7].clone()
        inp[k][-1, -1, j, 7] = v
        got = moda_attn_bwd(*args, O, LSE, inp["dO"])[0]
        inp[k][-1, -1, j, 7] = old
        G = Hq // Hk
        assert not torch.isfinite(got[-1, -G:, j:].float()).all(-1).any()
        got[-1, -G:, j - 5:] = clean[-1, -G:, j - 5:]
        assert torch.equal(got, clean)
