"""GPU parity of the backward on both sides of the rules that pick its dK/dV and dQ kernels by the
number of tiles: few tiles (32 keys or queries per workgroup, dealt out to its waves) and many (128 per
workgroup).  Bound and oracle as in test_bwd_parity."""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import synth
from test_bwd_parity import NAMES, check_full, compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 2, 3), (1, 2, 1, 31, 128, 5, None), (2, 2, 2, 32, 64, 6, None),
                                              (1, 4, 1, 33, 128, 3, 4), (1, 6, 2, 127, 64, 0, None), (1, 3, 3, 129, 128, 11, 12),
                                              (1, 10, 2, 161, 64, 4, None), (1, 9, 1, 97, 128, 2, None)])
def test_bwd_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    check_full(B, Hq, T, d, L, 1300 + T + L, causal=causal, depth_alloc=La, Hk=Hk)


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
