"""GPU parity: the decoding step (moda_attn_decode, through the C ABI) against the fp64 checker.

A decoding step is the operator at the last position of the attended prefix, so the checker's
row-sampled forward with rows = [T-1] is its definition; the depth cache of the step holds the
new token's slots only.  Tolerances: the forward's (2e-2 on O, 1e-3 on LSE, bf16 inputs)."""
import numpy as np
import pytest
import torch

from oracle import moda_ref as R
from paper_2603_15619_amd import synth

pytestmark = pytest.mark.gpu


def check(B, Hq, Hk, T, d, L, seed, kv_alloc=None, depth_alloc=None, scale=None):
    from paper_2603_15619_amd import moda_attn_decode

    kv_alloc = T if kv_alloc is None else kv_alloc
    La = L if depth_alloc is None else depth_alloc
    print("decode case", dict(B=B, Hq=Hq, Hk=Hk, T=T, d=d, L=L, kv_alloc=kv_alloc, depth_alloc=La, seed=seed), flush=True)
    # sequence cache of kv_alloc rows (the rows past T hold NaN: never attended);
    # one query row and one position's depth slots per sequence
    inp = synth.make_inputs(B, Hq, Hk, kv_alloc, d, 0, dtype="bf16", seed=seed, device="cuda")
    one = synth.make_inputs(B, Hq, Hk, 1, d, La, dtype="bf16", seed=seed + 1, device="cuda")
    Kc, Vc = inp["Kseq"], inp["Vseq"]
    Kc[:, :, T:] = float("nan")
    Vc[:, :, T:] = float("nan")
    Q = one["Q"][:, :, 0].contiguous()
    Kd = None if La == 0 else one["Kdepth"][:, :, 0].contiguous()
    Vd = None if La == 0 else one["Vdepth"][:, :, 0].contiguous()
    if La > L:
        Kd[:, :, L:] = float("nan")
        Vd[:, :, L:] = float("nan")
    O, LSE = moda_attn_decode(Q, Kc, Vc, Kd, Vd, T=T, depth_count=L, scale=scale)
    torch.cuda.synchronize()
    rows = np.array([T - 1], dtype=np.int32)
    f = synth.to_f64
    kd = None if La == 0 else np.nan_to_num(f(Kd))[:, :, None]
    vd = None if La == 0 else np.nan_to_num(f(Vd))[:, :, None]
    Oref, Lref = R.fwd_rows(f(Q)[:, :, None], f(Kc[:, :, :T]), f(Vc[:, :, :T]), kd, vd, rows, depth_count=L,
                            scale=scale)
    eo = np.abs(f(O) - Oref[:, :, 0]).max()
    el = np.abs(f(LSE) - Lref[:, :, 0]).max()
    print("   max|dO| = %.3e   max|dLSE| = %.3e" % (eo, el), flush=True)
    assert np.isfinite(f(O)).all() and eo <= 2e-2 and el <= 1e-3


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(2, 4, 4, 1000, 128, 15), (1, 8, 1, 777, 64, 5), (3, 6, 2, 300, 128, 0),
                                           (1, 16, 16, 5000, 128, 31), (2, 32, 2, 257, 64, 70), (1, 2, 2, 1, 128, 3),
                                           (1, 2, 1, 17, 64, 0), (4, 16, 8, 4096, 128, 15),
                                           # more than 4 heads per group: the matrix-pipe kernel (5 heads; 40 heads =
                                           # two chunks; the paper's kernel geometry on a long ragged cache; no slots)
                                           (1, 10, 2, 333, 128, 7), (1, 40, 1, 1500, 64, 33),
                                           (1, 64, 8, 20011, 64, 64), (2, 16, 2, 2049, 128, 0)])
def test_decode_shapes(B, Hq, Hk, T, d, L):
    check(B, Hq, Hk, T, d, L, 900 + T + L)


@pytest.mark.parametrize("seed", range(12))
def test_decode_random_shapes(seed):
    """Seeded random shapes: group sizes on both sides of the switch between the two partial
    kernels, ragged cache lengths, cache and slot strides larger than what is attended."""
    rng = np.random.default_rng(4200 + seed)
    d = int(rng.choice([64, 128]))
    Hk = int(rng.integers(1, 4))
    G = int(rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 33]))
    B = int(rng.integers(1, 4))
    T = int(rng.integers(1, 3000))
    L = int(rng.choice([0, 1, 5, 31, 32, 33, 100]))
    kv_alloc = T + int(rng.integers(0, 70))
    depth_alloc = L + int(rng.integers(0, 5))
    check(B, G * Hk, Hk, T, d, L, 4300 + seed, kv_alloc=kv_alloc, depth_alloc=depth_alloc)


def test_decode_cache_strides_and_scale():
    check(2, 4, 2, 500, 128, 3, 31, kv_alloc=1024, depth_alloc=8)
    check(1, 8, 8, 129, 64, 2, 32, kv_alloc=130, scale=0.3)
    check(1, 8, 1, 500, 64, 3, 36, kv_alloc=600, depth_alloc=8, scale=0.2)


def test_decode_long_cache():
    """B=2, H=16, T=65536: many slices per (batch, head)."""
    check(2, 16, 16, 65536, 128, 15, 33)


def test_decode_matches_last_row_of_prefill():
    """The step's output equals the last row of the full forward over the same prefix (within
    the forward's tolerance on both)."""
    from paper_2603_15619_amd import moda_attn_decode, moda_attn_fwd

    inp = synth.make_inputs(1, 4, 2, 700, 128, 6, dtype="bf16", seed=34, device="cuda")
    O, LSE = moda_attn_fwd(inp["Q"], inp["Kseq"], inp["Vseq"], inp["Kdepth"], inp["Vdepth"])
    Od, Ld = moda_attn_decode(inp["Q"][:, :, -1].contiguous(), inp["Kseq"], inp["Vseq"],
                              inp["Kdepth"][:, :, -1].contiguous(), inp["Vdepth"][:, :, -1].contiguous())
    torch.cuda.synchronize()
    assert (O[:, :, -1].float() - Od.float()).abs().max().item() <= 2e-2
    assert (LSE[:, :, -1] - Ld).abs().max().item() <= 1e-3


def test_decode_rejects_bad_arguments():
    from paper_2603_15619_amd import MODAError, moda_attn_decode

    inp = synth.make_inputs(1, 2, 2, 64, 128, 0, dtype="bf16", seed=35, device="cuda")
    q = inp["Q"][:, :, 0].contiguous()
    with pytest.raises(MODAError):
        moda_attn_decode(q, inp["Kseq"], inp["Vseq"], T=65)  # longer than the cache
    with pytest.raises(MODAError):
        moda_attn_decode(q, inp["Kseq"], inp["Vseq"], T=0)
    with pytest.raises(MODAError):
        moda_attn_decode(q.float(), inp["Kseq"].float(), inp["Vseq"].float())  # bf16 only


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(1, 4, 4, 1024, 128, 3), (1, 2, 2, 1025, 64, 0), (1, 8, 1, 2047, 64, 4),
                                           (1, 16, 2, 2176, 128, 5), (1, 8, 1, 128, 64, 0), (1, 1, 1, 40000, 64, 2)])
def test_decode_slice_counts(B, Hq, Hk, T, d, L):
    """Both sides of 8 slices of 128 keys, of one block per slice, and of the 16 slices up to which one
    group of threads folds a head."""
    check(B, Hq, Hk, T, d, L, 1900 + T)


def test_slices_fit_the_scratch_array_where_coarser_ones_do():
    """moda_attn_decode_noalloc takes what 256-key slices would let it take (the first three: 128-key slices, of
    every (batch, head) and with the depth slots' slice, would not fit)."""
    import ctypes

    from paper_2603_15619_amd.binding import MODAShape, lib

    most = lib().moda_attn_decode_noalloc_max_bytes()
    for B, Hk, G, T, d in [(8, 8, 8, 4000, 128), (8, 16, 8, 2000, 128), (1, 16, 16, 16000, 64)]:
        one = B * G * Hk * (d + 2) * 4
        assert ((T + 127) // 128 + 1) * one > most >= ((T + 255) // 256 + 1) * one
        s = MODAShape(B, G * Hk, Hk, T, d, 2, 2, 1, 0.0, 1)
        assert lib().moda_attn_decode_workspace_bytes(ctypes.byref(s)) <= most
    for B, Hk, G, T, d in [(8, 2, 32, 2000, 128), (30, 1, 8, 16000, 64), (400, 4, 1, 1000, 128), (6, 1, 64, 5000, 64)]:
        s = MODAShape(B, G * Hk, Hk, T, d, 2, 2, 1, 0.0, 1)
        coarse = B * G * Hk * ((T + 255) // 256 + 1) * (d + 2) * 4
        if coarse <= most:
            assert lib().moda_attn_decode_workspace_bytes(ctypes.byref(s)) <= most


@pytest.mark.parametrize("B,Hq,Hk,d,T_max,calls", [(8, 64, 8, 64, 8192, [(8, 4097), (8, 6000), (8, 7808)]),
                                                   (8, 64, 8, 128, 4096, [(8, 2049), (8, 3840), (7, 4096), (4, 4096)]),
                                                   (12, 8, 8, 64, 3000, [(12, 1999), (5, 3000), (1, 1001)])])
def test_one_workspace_for_a_serving_loop(B, Hq, Hk, d, T_max, calls):
    """A workspace sized once, for the largest batch at its longest context, serves every call of the loop, and
    the results are those of a call with a workspace of its own (both to the forward's tolerance)."""
    import ctypes

    from paper_2603_15619_amd import moda_attn_decode
    from paper_2603_15619_amd.binding import MODAShape, lib

    size = lib().moda_attn_decode_workspace_bytes(ctypes.byref(MODAShape(B, Hq, Hk, T_max, d, 3, 3, 1, 0.0, 1)))
    for b, T in calls:
        inp = synth.make_inputs(b, Hq, Hk, T, d, 0, dtype="bf16", seed=2000 + T, device="cuda")
        one = synth.make_inputs(b, Hq, Hk, 1, d, 3, dtype="bf16", seed=2001 + T, device="cuda")
        args = [one["Q"][:, :, 0].contiguous(), inp["Kseq"], inp["Vseq"], *(one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))]
        both = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device="cuda")  # (nothing is written past the workspace)
        O, LSE = moda_attn_decode(*args, workspace=both[:size])
        O1, LSE1 = moda_attn_decode(*args)
        torch.cuda.synchronize()
        assert (both[size:] == 0x5a).all()
        assert (O.float() - O1.float()).abs().max().item() <= 2e-2 and (LSE - LSE1).abs().max().item() <= 1e-3


@pytest.mark.parametrize("B,Hq,Hk,T,d,lo,hi", [(1, 2, 2, 8192, 64, 512, 8192), (2, 4, 2, 9000, 128, 0, 8000), (1, 1, 1, 700, 64, 128, 256),
                                               (1, 8, 1, 1003, 64, 128, 160), (1, 16, 2, 5000, 128, 96, 4900)])
def test_decode_keys_of_weight_zero(B, Hq, Hk, T, d, lo, hi):
    """Keys whose scores are -inf weigh nothing, also where a block, a slice or a group of slices holds no
    other: the result is that of a cache without them (to the forward's tolerance, both sides)."""
    from paper_2603_15619_amd import moda_attn_decode

    inp = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2200 + T, device="cuda")
    K, V, Q = inp["Kseq"], inp["Vseq"], inp["Q"][:, :, 0].abs().contiguous() + 0.1  # (positive: -inf, not NaN)
    keep = [t for t in range(T) if t < lo or t >= hi]
    O1, LSE1 = moda_attn_decode(Q, K[:, :, keep].contiguous(), V[:, :, keep].contiguous())
    K[:, :, lo:hi] = -float("inf")
    O, LSE = moda_attn_decode(Q, K, V)
    torch.cuda.synchronize()
    assert (O.float() - O1.float()).abs().max().item() <= 2e-2
    assert (LSE - LSE1).abs().max().item() <= 1e-3


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,slices", [(4, 16, 8, 1500, 128, 12, 6), (3, 16, 8, 1500, 128, 12, 8), (1, 16, 16, 1003, 128, 2, 8),
                                                  (36, 2, 2, 1271, 64, 7, 5), (1, 4, 4, 1024, 64, 1, 8), (1, 4, 4, 1025, 64, 1, 5),
                                                  (1, 4, 4, 1536, 128, 1, 8), (1, 4, 4, 1537, 128, 1, 7), (64, 2, 2, 281, 128, 3, 3), (64, 2, 2, 281, 128, 0, 2),
                                                  (23, 128, 16, 430, 64, 1, 2), (16, 128, 16, 380, 64, 4, 3),
                                                  (16, 128, 16, 470, 64, 4, 2), (16, 128, 16, 470, 128, 4, 4)])
def test_finer_slices_only_where_they_make_no_more_rounds(B, Hq, Hk, T, d, L, slices):
    """The partial results that a call writes tell its slices: of at most 256 keys, or finer ones where these
    leave no more workgroups than rounds of 256 (512 for groups of more than 4 heads at d = 128) hold already, up to
    8 of them for groups of up to 4 heads."""
    from paper_2603_15619_amd import moda_attn_decode

    one = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2300, device="cuda")
    seq = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2301, device="cuda")
    kd, vd = (None if L == 0 else one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    ws = torch.full((B * Hq * 20 * (d + 2),), float("nan"), device="cuda")
    moda_attn_decode(one["Q"][:, :, 0].contiguous(), seq["Kseq"], seq["Vseq"], kd, vd, workspace=ws)
    torch.cuda.synchronize()
    written = int((~torch.isnan(ws)).sum().item())
    assert written == B * Hq * (slices + (L > 0)) * (d + 2)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,slices", [(1, 8, 1, 512, 64, 0, 16), (1, 8, 1, 513, 64, 3, 9), (1, 16, 2, 129, 128, 1, 5), (6, 64, 8, 512, 128, 0, 16),
                                                  (7, 64, 8, 500, 128, 2, 8), (1, 8, 1, 6144, 64, 0, 96), (1, 8, 1, 6145, 64, 0, 49),
                                                  (1, 4, 4, 512, 128, 1, 8), (1, 4, 4, 513, 128, 1, 5), (9, 3, 3, 300, 128, 0, 5), (1, 4, 4, 1793, 128, 0, 29),
                                                  (1, 4, 4, 2048, 128, 5, 32), (1, 4, 4, 2049, 128, 5, 17), (1, 4, 4, 1792, 64, 2, 7), (1, 4, 2, 1793, 64, 2, 15),
                                                  (1, 2, 2, 4096, 64, 1, 32), (1, 2, 2, 4097, 64, 1, 17), (3, 16, 4, 3000, 128, 4, 12),
                                                  # 32 heads per workgroup; two slices of 32 keys beside 32 and 33 slots
                                                  (4, 64, 2, 300, 64, 0, 10), (5, 64, 2, 300, 64, 0, 5), (4, 64, 2, 1000, 64, 3, 16), (16, 128, 4, 512, 64, 1, 8), (17, 128, 4, 378, 64, 7, 6),
                                                  (16, 64, 4, 256, 128, 0, 8), (17, 64, 4, 256, 128, 0, 4), (3, 64, 1, 512, 128, 2, 16),
                                                  (130, 8, 1, 43, 64, 32, 2), (130, 8, 1, 43, 64, 33, 1), (130, 8, 1, 43, 128, 64, 1)])
def test_finest_slices_of_calls_with_few_workgroups(B, Hq, Hk, T, d, L, slices):
    """Slices of 32 and 64 keys (groups of more than 4 heads), of 64 and 128 (others), where their workgroups leave
    units over, and the next coarser ones beyond."""
    from paper_2603_15619_amd import moda_attn_decode
    from paper_2603_15619_amd.binding import MODAShape, lib
    import ctypes

    one = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2400, device="cuda")
    seq = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2401, device="cuda")
    kd, vd = (None if L == 0 else one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    size = lib().moda_attn_decode_workspace_bytes(ctypes.byref(MODAShape(B, Hq, Hk, T, d, L, L, 1, 0.0, 1)))
    ws = torch.full((size // 4 + 1000,), float("nan"), device="cuda")
    moda_attn_decode(one["Q"][:, :, 0].contiguous(), seq["Kseq"], seq["Vseq"], kd, vd, workspace=ws[:size // 4])
    torch.cuda.synchronize()
    assert int((~torch.isnan(ws)).sum().item()) == B * Hq * (slices + (L > 0)) * (d + 2)
    check(B, Hq, Hk, T, d, L, 2402)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 0, 0), (1, 2, 2, 1, 128, 3, 4), (2, 4, 4, 255, 64, 1, None), (3, 4, 4, 257, 64, 0, 2), (1, 3, 3, 700, 64, 67, 70),
                                              (5, 4, 4, 127, 128, 1, None), (2, 2, 2, 129, 128, 0, None), (3, 2, 2, 200, 128, 56, 60), (40, 16, 8, 100, 64, 7, None), (2, 4, 2, 480, 64, 31, 33),
                                              (3, 4, 2, 250, 128, 5, None), (4, 8, 2, 250, 64, 6, 7), (2, 6, 2, 96, 128, 32, None), (7, 4, 1, 31, 128, 0, None), (33, 16, 16, 400, 128, 15, 16),
                                              (3, 8, 1, 200, 64, 56, None), (2, 10, 2, 100, 128, 15, 17), (1, 64, 1, 128, 128, 0, None), (1, 13, 1, 17, 64, 0, 1)])
def test_short_contexts_take_one_kernel(B, Hq, Hk, T, d, L, La):
    """Keys and slots of few batches: nothing is written to the workspace; rows past T in the cache and slots past L hold NaN."""
    from paper_2603_15619_amd import moda_attn_decode

    La = L if La is None else La
    one = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2500 + T, device="cuda", depth_alloc=La)
    seq = synth.make_inputs(B, Hq, Hk, T + 3, d, 0, dtype="bf16", seed=2501 + T, device="cuda")
    K, V = seq["Kseq"], seq["Vseq"]
    K[:, :, T:] = float("nan")
    V[:, :, T:] = float("nan")
    kd, vd = (None if La == 0 else one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    if La > L:
        kd[:, :, L:] = float("nan")
        vd[:, :, L:] = float("nan")
    Q = one["Q"][:, :, 0].contiguous()
    ws = torch.full((1 << 22,), float("nan"), device="cuda")
    O, LSE = moda_attn_decode(Q, K, V, kd, vd, T=T, depth_count=L, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isnan(ws).all()
    f = lambda t: synth.to_f64(t)  # noqa: E731
    Oref, Lref = R.fwd_rows(f(Q)[:, :, None], f(K[:, :, :T].contiguous()), f(V[:, :, :T].contiguous()),
                            None if L == 0 else f(kd[:, :, :L].contiguous())[:, :, None], None if L == 0 else f(vd[:, :, :L].contiguous())[:, :, None],
                            np.array([T - 1], dtype=np.int32), depth_count=L)
    assert np.abs(f(O) - Oref[:, :, 0]).max() <= 2e-2 and np.abs(f(LSE) - Lref[:, :, 0]).max() <= 1e-3


def test_more_heads_than_one_kernel_has_workgroups():
    """2^23 + 8 heads: too many workgroups of eight waves for one launch, so two kernels take the call.  One key has
    weight 1: O is V."""
    from paper_2603_15619_amd import moda_attn_decode

    Q = torch.zeros(((1 << 20) + 1, 8, 64), dtype=torch.bfloat16, device="cuda")
    V = torch.randn(Q.shape, dtype=torch.bfloat16, device="cuda")[:, :, None]
    O, LSE = moda_attn_decode(Q, Q[:, :, None], V)
    assert torch.equal(O, V[:, :, 0]) and torch.count_nonzero(LSE) == 0


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(1, 2, 2, 128, 64, 0), (2, 2, 1, 256, 64, 0), (1, 4, 1, 128, 128, 0), (1, 8, 1, 100, 64, 0), (1, 1, 1, 33, 128, 0),
                                           (3, 2, 2, 200, 64, 5), (1, 3, 1, 1, 64, 1)])
def test_infinite_value_of_the_last_row(B, Hq, Hk, T, d, L):
    """Short contexts: the last key (or slot) has an infinite value in two channels; its weight is positive, so the
    output is infinite there, with its sign, and what it was everywhere else."""
    from paper_2603_15619_amd import moda_attn_decode

    one = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2600, device="cuda")
    seq = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2601, device="cuda")
    kd, vd = (None if L == 0 else one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    args = [one["Q"][:, :, 0].contiguous(), seq["Kseq"], seq["Vseq"], kd, vd]
    O, LSE = moda_attn_decode(*args)
    last = seq["Vseq"] if L == 0 else vd
    last[:, :, -1, 3] = float("inf")
    last[:, :, -1, d - 1] = -float("inf")
    Oinf, LSEinf = moda_attn_decode(*args)
    assert (Oinf[..., 3] == float("inf")).all() and (Oinf[..., d - 1] == -float("inf")).all()
    keep = [c for c in range(d) if c not in (3, d - 1)]
    assert torch.equal(Oinf[..., keep], O[..., keep]) and torch.equal(LSEinf, LSE)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L", [(33, 64, 2, 1100, 64, 3), (17, 64, 2, 1300, 128, 0), (32, 64, 2, 1100, 64, 3), (257, 8, 2, 2304, 64, 0)])
def test_merge_of_9_to_16_slices_on_both_sides_of_2_to_the_17_outputs(B, Hq, Hk, T, d, L):
    check(B, Hq, Hk, T, d, L, 2700)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,one", [(256, 3, 1, 12, 64, 0, True), (257, 3, 1, 12, 64, 0, False), (257, 4, 1, 12, 64, 3, True), (64, 32, 8, 49, 128, 7, True),
                                               (513, 4, 1, 12, 64, 3, False), (65, 24, 8, 49, 128, 7, False), (33, 16, 8, 979, 64, 7, False), (48, 16, 8, 979, 64, 7, True),
                                               (33, 8, 8, 760, 64, 0, True)])
def test_one_kernel_above_256_workgroups(B, Hq, Hk, T, d, L, one):
    """Groups of 3 and 4 heads: only up to 512 workgroups and with a second slice; others: up to three batches of rows,
    and four from 384 workgroups on.  The kernel writes nothing to the workspace."""
    from paper_2603_15619_amd import moda_attn_decode

    tok = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2800, device="cuda")
    seq = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2801, device="cuda")
    kd, vd = (None if L == 0 else tok[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    ws = torch.full((1 << 23,), float("nan"), device="cuda")
    moda_attn_decode(tok["Q"][:, :, 0].contiguous(), seq["Kseq"], seq["Vseq"], kd, vd, workspace=ws)
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws).all()) == one
    check(B, Hq, Hk, T, d, L, 2802)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,row", [(2, 4, 4, 1000, 128, 1, None), (3, 4, 2, 700, 64, 2, None), (1, 4, 1, 600, 64, 1, None), (2, 3, 3, 513, 128, 0, 512),
                                               (2, 16, 2, 1000, 64, 1, None), (2, 4, 2, 100, 64, 1, None), (1, 2, 2, 65, 128, 0, 64), (1, 4, 4, 1, 64, 0, 0)])
def test_nan_key_is_not_lost(B, Hq, Hk, T, d, L, row):
    """A key (or, row None, the last slot) of the last sequence's last head is NaN, alone in its lanes' share of the rows:
    the outputs of its query heads are NaN, the others what they were."""
    from paper_2603_15619_amd import moda_attn_decode

    one = synth.make_inputs(B, Hq, Hk, 1, d, L, dtype="bf16", seed=2900, device="cuda")
    seq = synth.make_inputs(B, Hq, Hk, T, d, 0, dtype="bf16", seed=2901, device="cuda")
    kd, vd = (None if L == 0 else one[k][:, :, 0].contiguous() for k in ("Kdepth", "Vdepth"))
    args = [one["Q"][:, :, 0].contiguous(), seq["Kseq"], seq["Vseq"], kd, vd]
    O, LSE = (x.view(B, Hk, Hq // Hk, -1).clone() for x in moda_attn_decode(*args))
    (kd if row is None else seq["Kseq"])[-1, -1, -1 if row is None else row, 5] = float("nan")
    On, LSEn = (x.view(B, Hk, Hq // Hk, -1) for x in moda_attn_decode(*args))
    assert torch.isnan(On[-1, -1]).all() and torch.isnan(LSEn[-1, -1]).all()
    On[-1, -1], LSEn[-1, -1] = O[-1, -1], LSE[-1, -1]
    assert torch.equal(On, O) and torch.equal(LSEn, LSE)
