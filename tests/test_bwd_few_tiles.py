"""GPU parity of the backward on both sides of the rules that pick its kernels by the
number of tiles: few tiles (32 keys or queries per workgroup, dealt out to its waves) and many (128 per
workgroup), in the dK/dV and dQ kernels (groups of 3, 5 and more heads with slots, or up to 16 positions) and in
the kernel of all three gradients.  Bound and oracle as in test_bwd_parity."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import moda_attn_bwd, moda_attn_fwd, synth
from paper_2603_15619_amd.binding import MODAShape, lib
from test_bwd_parity import NAMES, check_full, compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 2, 3), (1, 2, 1, 31, 128, 5, None), (2, 2, 2, 32, 64, 6, None),
                                              (1, 4, 1, 33, 128, 3, 4), (1, 6, 2, 127, 64, 0, None), (1, 3, 3, 129, 128, 11, 12),
                                              (1, 10, 2, 161, 64, 4, None), (1, 9, 1, 97, 128, 2, None)])
def test_bwd_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    check_full(B, Hq, T, d, L, 1300 + T + L, causal=causal, depth_alloc=La, Hk=Hk)


def kernel(B, Hq, Hk, T, d, L, causal, which, La=None):
    """The kernel of dK and dV (which = 0) or of dQ (1)."""
    s = MODAShape(B, Hq, Hk, T, d, L if La is None else La, L, int(causal), 0.0, 1)
    name = ctypes.create_string_buffer(64)
    lib().moda_bwd_kernel_name(ctypes.byref(s), which, name, len(name))
    return name.value.decode()


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", [(1, 8, 1, 777, 0, None, True), (1, 6, 2, 1500, 4, 5, True),
                                                   (1, 4, 2, 1100, 7, None, True), (1, 3, 3, 2050, 5, 6, True), (2, 10, 1, 333, 2, None, False),
                                                   (1, 8, 2, 1001, 24, None, False), (1, 8, 1, 97, 0, None, True), (3, 8, 1, 33, 9, 10, True)])
def test_bwd_few_tiles_of_many_queries(B, Hq, Hk, T, L, La, causal):
    """d = 64, few key tiles that see many queries: eight waves per key tile, in the dK/dV kernel or in one launch."""
    assert kernel(B, Hq, Hk, T, 64, L, causal, 0, La).endswith(", 8>")
    check_full(B, Hq, T, 64, L, 1350 + T + L, causal=causal, depth_alloc=La, Hk=Hk)


def check_ends(B, Hq, Hk, T, d, L, seed, causal):
    """The first and the last sequence (they differ in their data only)."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=seed, device="cuda", with_dO=True)
    grads = run_gpu(inp, L, causal)
    for b in {0, B - 1}:
        args = [None if inp[k] is None else synth.to_f64(inp[k][b:b + 1]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth", "dO")]
        ref, noise = R.bwd(*args, depth_count=L, causal=causal), R.bwd_noise(*args, depth_count=L, causal=causal)
        for name, g, r, n in zip(NAMES, grads, ref, noise):
            if g is not None:
                compare(name, g[b:b + 1], r, n)
    for g in grads:
        assert g is None or torch.isfinite(g.float()).all()


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(5, 39, 13, 610, 128, 2), (51, 9, 3, 300, 64, 2), (1, 15, 5, 3300, 64, 2), (1, 21, 7, 2100, 128, 1)])
def test_bwd_grids_of_one_round(B, Hq, Hk, T, d, L):
    """Between one and two workgroups per compute unit in the dK/dV kernel of 128 keys (the first two) or in the dQ kernel of 128
    queries, a number that 8 does not divide: tiles of every other layer in reverse."""
    names = [kernel(B, Hq, Hk, T, d, L, True, which) for which in (0, 1)]
    grids = [B * H * -(-T // 128) for n, H in zip(names, (Hk, Hq)) if n.startswith(("moda_bwd_dkdv_kernel", "moda_bwd_dq_kernel"))]
    assert any(256 < g <= 512 and g % 8 != 0 for g in grids)
    check_ends(B, Hq, Hk, T, d, L, 1380 + T, True)


@pytest.mark.parametrize("B,Hq,T,d,L", [(3, 11, 1600, 128, 0), (1, 23, 2500, 64, 2), (5, 13, 610, 128, 3)])
def test_bwd_heads_that_8_does_not_divide(B, Hq, T, d, L):
    """One launch for all three gradients, heads walked tile by tile over all dies."""
    assert "grads" in kernel(B, Hq, Hq, T, d, L, True, 0)
    check_ends(B, Hq, Hq, T, d, L, 1380 + T, True)


@pytest.mark.parametrize("B,Hq,Hk,T,L,causal", [(65, 24, 8, 33, 2, True), (75, 10, 2, 127, 1, False), (37, 30, 6, 321, 1, True), (23, 6, 2, 400, 2, True),
                                                (8, 40, 8, 1100, 1, False), (13, 15, 5, 300, 2, True), (70, 24, 8, 400, 1, True)])
def test_bwd_three_workgroups_per_unit(B, Hq, Hk, T, L, causal):
    """d = 64, the dQ kernel's grids that take three workgroups per compute unit: short sequences, one
    round of three (in layers where causal; 8 does not divide it), many workgroups."""
    assert kernel(B, Hq, Hk, T, 64, L, causal, 1) == "moda_bwd_dq_kernel<64, 4, 3>"
    check_ends(B, Hq, Hk, T, 64, L, 1390 + T, causal)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(89, 8, 8, 130, 64, 5, 6, True), (89, 16, 8, 131, 64, 3, None, True),
                                                     (45, 32, 8, 190, 64, 2, 3, True), (24, 16, 8, 257, 128, 6, None, False),
                                                     (24, 64, 16, 65, 128, 1, 2, True), (24, 40, 8, 130, 64, 2, None, False)])
def test_bwd_many_tiles_of_short_sequences(B, Hq, Hk, T, d, L, La, causal):
    """Enough (batch, head) pairs for the kernels of 128 keys / queries per workgroup."""
    check_full(B, Hq, T, d, L, 1400 + T + L, causal=causal, depth_alloc=La, Hk=Hk)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(89, 64, 8, 130, 64, 20, 21, True), (89, 40, 8, 129, 64, 32, None, True),
                                                     (45, 48, 8, 255, 64, 47, 50, False), (24, 56, 8, 257, 128, 28, 30, False),
                                                     (24, 64, 8, 200, 128, 64, None, True)])
def test_bwd_depth_slots_of_5_to_8_heads_inside_dkdv(B, Hq, Hk, T, d, L, La, causal):
    """Groups of 5 to 8 heads with well-filled blocks of 32 slots: the depth-slot gradients run inside
    the dK/dV kernel on the matrix pipe; unattended slots hold NaN and get zero gradients."""
    inp = synth.make_inputs(B, Hq, Hk, T, d, L, dtype="bf16", seed=1800 + T + L, device="cuda", depth_alloc=La, with_dO=True)
    if La is not None:
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    grads = run_gpu(inp, L, causal)
    # the first and the last sequence in full; the others only differ in their data
    for b in (slice(0, 1), slice(B - 1, B)):
        args = [np.nan_to_num(synth.to_f64(inp[k][b])) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth", "dO")]
        ref = R.bwd(*args, depth_count=L, causal=causal)
        noise = R.bwd_noise(*args, depth_count=L, causal=causal)
        for name, g, r, n in zip(NAMES, grads, ref, noise):
            compare(name, g[b], r, n)
    for g in grads:
        assert torch.isfinite(g.float()).all()


def inside_dkdv(B, Hq, Hk, T, L, causal):
    s = MODAShape(B, Hq, Hk, T, 64, L, L, int(causal), 0.0, 1)
    return lib().moda_kernels_per_call(ctypes.byref(s), 1) == 3


@pytest.mark.parametrize("B,Hq,Hk,T,L,La,causal", [(9, 64, 8, 512, 32, None, False), (24, 40, 8, 530, 47, 50, True),
                                                   (13, 56, 8, 600, 28, 30, False), (16, 64, 8, 635, 56, None, True)])
def test_bwd_depth_slots_inside_dkdv(B, Hq, Hk, T, L, La, causal):
    """As above at sizes that take the combined kernel."""
    assert inside_dkdv(B, Hq, Hk, T, L, causal)
    inp = synth.make_inputs(B, Hq, Hk, T, 64, L, dtype="bf16", seed=1900 + T + L, device="cuda", depth_alloc=La, with_dO=True)
    if La is not None:
        inp["Kdepth"][:, :, :, L:] = float("nan")
        inp["Vdepth"][:, :, :, L:] = float("nan")
    grads = run_gpu(inp, L, causal)
    args = [np.nan_to_num(synth.to_f64(inp[k][B - 1:])) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth", "dO")]
    ref, noise = R.bwd(*args, depth_count=L, causal=causal), R.bwd_noise(*args, depth_count=L, causal=causal)
    for name, g, r, n in zip(NAMES, grads, ref, noise):
        compare(name, g[B - 1:], r, n)
    for g in grads:
        assert torch.isfinite(g.float()).all()


def test_depth_gradients_of_8_heads_use_32_bit_weights():
    """Two heads whose weights on a slot differ by some 2^-14 of them and whose dO are opposite: dVdepth is that
    difference.  Each weight is 2^(s - lse) with both terms below 16 and rounded at 2^-21, an error of the
    difference of 2^-20.5 of the weight at most (twice 2^-21 ln 2); the bf16 result,
    2^-14 of it, adds 2^-23.  Weights of 16 bits were off by 2^-18.4."""
    B, Hk, G, T, L, d = 9, 8, 8, 512, 32, 64
    assert inside_dkdv(B, G * Hk, Hk, T, L, False)
    inp = synth.make_inputs(B, G * Hk, Hk, T, d, L, dtype="bf16", seed=77, device="cuda", with_dO=True)
    for k in ("Q", "Kseq", "Kdepth"):
        inp[k] *= 0.25
    inp["Kseq"][..., 0] = 0.0
    inp["Kdepth"][..., 0] = 2.0 ** -12  # times a difference of 2 in Q's first channel, scaled by 1 / 8 ...
    inp["Kdepth"][:, :, :, ::2, 0] *= -1  # ... up or down (a common shift would cancel in the weights)
    Q, dO = (inp[k].view(B, Hk, G, T, d) for k in ("Q", "dO"))
    Q[:, :, 1] = Q[:, :, 0]
    Q[:, :, 0, :, 0], Q[:, :, 1, :, 0] = 1.0, -1.0
    dO.zero_()
    dO[:, :, 0], dO[:, :, 1] = 1.0, -1.0
    args = [inp[n] for n in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")]
    O, _ = moda_attn_fwd(*args, causal=False)
    LSE = torch.empty(B, G * Hk, T, device="cuda")
    P = torch.empty(B, Hk, 2, T, L, dtype=torch.float64, device="cuda")  # weights of the first two heads
    for b in range(B):
        for g in range(Hk):
            q, k, kd = Q[b, g].double(), inp["Kseq"][b, g].double(), inp["Kdepth"][b, g].double()
            sd = (kd[None] * q[:, :, None]).sum(-1) / 8
            lse = torch.logsumexp(torch.cat([(q.reshape(-1, d) @ k.t().contiguous()).view(G, T, T) / 8, sd], -1), -1)
            LSE[b, g * G:(g + 1) * G] = lse.float()  # (its rounding is no part of the kernel's error)
            P[b, g] = torch.exp(sd - LSE[b, g * G:(g + 1) * G].double()[..., None])[:2]
    dVd = moda_attn_bwd(*args, O, LSE, inp["dO"], causal=False)[4].double()
    ref = (P[:, :, 0] - P[:, :, 1])[..., None].expand_as(dVd)
    rms = ((dVd - ref) / P[:, :, 0, :, :, None]).square().mean().sqrt().item()
    print("rms error of the difference over the weight: 2^%.2f" % np.log2(rms), flush=True)
    assert rms <= 2.0 ** -20.5


@pytest.mark.parametrize("B,T,L,causal", [(9, 512, 32, False), (16, 635, 48, True)])
def test_infinite_dO_of_8_heads_stays_infinite(B, T, L, causal):
    """An infinite element of dO: dVdepth is infinite in that channel of that position (every weight is
    positive), one bf16 rounding off at most in the others (another order of fp32 sums), and no other
    position's depth gradients change."""
    assert inside_dkdv(B, 64, 8, T, L, causal)
    inp = synth.make_inputs(B, 64, 8, T, 64, L, dtype="bf16", seed=78, device="cuda", with_dO=True)
    clean = run_gpu(inp, L, causal)
    b, h, t, c = 3, 2, T // 2, 5
    inp["dO"][b, h, t, c] = -float("inf")
    grads = run_gpu(inp, L, causal)
    at = (b, h // 8, t)
    assert (grads[4][at][:, c] == -float("inf")).all()
    others = [i for i in range(64) if i != c]
    x, y = (g[4][at][:, others].float() for g in (grads, clean))
    assert ((x - y).abs() <= 2.0 ** -7 * y.abs() + 2.0 ** -20).all()
    for g, k in zip(grads[3:], clean[3:]):
        g[at] = k[at]
        assert torch.equal(g, k)
