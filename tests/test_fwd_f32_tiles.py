"""GPU parity of the fp32 forward at the edges of its tiles (32 queries x 32 keys, key tiles dealt
to 4 waves, depth slots in chunks of 3 or 6): against the fp64 oracle, through the C ABI.

Tolerance 1e-5 (max abs): |O| <= 5 here and a weight or an output is a sum of at most a few hundred
terms rounded at 2^-24 relative, an error of some 1e-6 at most."""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import moda_attn_fwd, synth

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


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("T,d,at", [(70, 64, 37), (130, 128, 129), (64, 128, 0)])
def test_f32_value_that_is_not_finite_stays_behind_the_diagonal(T, d, at, value):
    """A value row that is infinite or NaN reaches the queries that see it and no other, those that
    share its tile with a weight of zero among them."""
    O, LSE, (Oref, Lref) = run(1, 2, 1, T, d, 2, 90 + T, spoil=(at, value))
    assert np.abs(LSE - Lref).max() <= TOL
    if at:
        assert np.abs(O[:, :, :at] - Oref[:, :, :at]).max() <= TOL
    assert not np.isfinite(O[:, :, at:]).any()
