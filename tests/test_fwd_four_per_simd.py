"""GPU parity of the bf16 forward at d = 64 in grids large enough for four waves per SIMD (steps of half a key
tile): lengths around tiles and half tiles, grids of one round with a last layer of workgroups that is not
full, both workgroup sizes, scores that jump.  Against the fp64 oracle on the first and the last batch element;
tolerances as in test_fwd_parity, for scores that jump as in test_fwd_reference_raise."""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import synth
from test_fwd_parity import run_gpu

pytestmark = pytest.mark.gpu


def against_oracle(inp, B, L, causal, O, LSE, tol_o, tol_l):
    for b in (0, B - 1):
        one = {k: None if v is None else v[b:b + 1].contiguous() for k, v in inp.items()}
        Oref, Lref = R.fwd(*(synth.to_f64(one[k]) for k in ("Q", "Kseq", "Vseq", "Kdepth", "Vdepth")),
                           depth_count=L, causal=causal)
        assert np.abs(synth.to_f64(O[b:b + 1]) - Oref).max() <= tol_o(one)
        assert (np.abs(synth.to_f64(LSE[b:b + 1]) - Lref) <= tol_l(Lref)).all()


@pytest.mark.parametrize("waves", [0, 4, 8])
@pytest.mark.parametrize("B,Hq,Hk,T,L,causal", [
    (40, 16, 16, 1, 2, True), (35, 16, 16, 31, 0, True), (33, 16, 16, 33, 4, True), (20, 32, 8, 64, 5, False),
    (30, 20, 20, 65, 0, False), (9, 32, 16, 161, 7, True), (9, 9, 9, 1000, 0, True), (11, 7, 7, 1000, 3, True),
    (5, 24, 3, 710, 12, True), (37, 5, 5, 417, 1, False), (13, 16, 16, 930, 2, True)])
def test_large_grids(B, Hq, Hk, T, L, causal, waves):
    print("case", B, Hq, Hk, T, L, causal, waves, flush=True)
    inp = synth.make_inputs(B, Hq, Hk, T, 64, L, dtype="bf16", seed=2000 + T, device="cuda")
    O, LSE = run_gpu(inp, L, causal, tuning=dict(waves=waves) if waves else None)
    against_oracle(inp, B, L, causal, O, LSE, lambda _: 2e-2, lambda _: 1e-3)


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("Hk,T,L,causal", [(4, 580, 0, True), (2, 650, 6, True), (4, 390, 5, False)])
def test_scores_that_jump(waves, Hk, T, L, causal):
    B, Hq = 50, 4  # (more than 512 workgroups of 4 waves)
    inp = synth.make_inputs(B, Hq, Hk, T, 64, L, dtype="bf16", seed=2100 + T, device="cuda")
    for pos, factor in ((0, 8.0), (31, 20.0), (32, 40.0), (63, 60.0), (100, 200.0), (130, 250.0), (225, 300.0),
                        (290, 350.0), (T - 33, 380.0), (T - 1, 400.0)):
        inp["Kseq"][:, :, pos] *= factor
    O, LSE = run_gpu(inp, L, causal, tuning=dict(waves=waves))
    assert torch.isfinite(O.float()).all() and torch.isfinite(LSE).all()
    vmax = lambda one: 2 * 2.0 ** -8 * max(float(one[k].abs().max()) for k in (("Vseq", "Vdepth") if L else ("Vseq",)))
    against_oracle(inp, B, L, causal, O, LSE, vmax, lambda ref: 1e-3 + 4 * 2.0 ** -24 * np.abs(ref))
