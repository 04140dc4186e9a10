"""Host-only checks of the C ABI: the library loads, exports every symbol the
header declares, and rejects bad shapes before touching a GPU."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "moda.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(moda_[a-z_0-9]+)\s*\(", text)))


@pytest.fixture(scope="module")
def L():
    from paper_2603_15619_amd import binding as libmoda

    if not os.path.exists(libmoda.LIB_PATH):
        from paper_2603_15619_amd.build import build_libmoda

        build_libmoda()
    return libmoda.lib()


def test_header_functions_are_exported(L):
    names = declared_functions()
    assert {"moda_attn_fwd", "moda_attn_bwd", "moda_attn_bwd_workspace_bytes",
            "moda_status_string", "moda_version"} <= set(names)
    for n in names:
        assert hasattr(L, n), n


def test_binding_lists_every_export():
    from paper_2603_15619_amd import binding as libmoda

    assert sorted(libmoda.EXPORTS) == declared_functions()


def test_status_strings_and_version(L):
    from paper_2603_15619_amd import binding as libmoda

    assert L.moda_version() >= 100
    seen = {libmoda.status_string(c) for c in range(7)}
    assert len(seen) == 7 and "ok" in seen


def test_shape_errors_without_gpu(L):
    from paper_2603_15619_amd.binding import MODAShape

    def fwd(shape, ptr=0x1000):
        p = ctypes.c_void_p(ptr)
        return L.moda_attn_fwd(p, p, p, p, p, p, p, ctypes.byref(shape), None)

    ok = dict(B=1, Hq=2, Hk=2, T=16, d=128, depth_alloc=2, depth_count=2, causal=1, scale=0.0, dtype=1)
    assert L.moda_attn_fwd(None, None, None, None, None, None, None, None, None) == 1  # NULL shape
    assert fwd(MODAShape(**dict(ok, d=96))) == 3          # unsupported head dim
    assert fwd(MODAShape(**dict(ok, dtype=7))) == 3       # unsupported dtype
    assert fwd(MODAShape(**dict(ok, Hq=3))) == 2          # Hq % Hk != 0
    assert fwd(MODAShape(**dict(ok, depth_count=3))) == 2  # more slots than allocated
    assert fwd(MODAShape(**dict(ok, T=-1))) == 2
    assert fwd(MODAShape(**dict(ok, causal=2))) == 2
    assert fwd(MODAShape(**ok), ptr=0x1008) == 4          # misaligned pointer
    assert L.moda_attn_fwd(None, None, None, None, None, None, None,
                           ctypes.byref(MODAShape(**ok)), None) == 1  # NULL tensors
    assert fwd(MODAShape(**dict(ok, B=0))) == 0           # empty problem: nothing launched
    assert fwd(MODAShape(**dict(ok, T=0))) == 0


def test_new_entry_points_reject_bad_arguments_without_gpu(L):
    """moda_depth_append, moda_attn_decode and moda_attn_bwd validate everything on the host
    before any kernel is launched."""
    from paper_2603_15619_amd.binding import MODAShape

    ok = dict(B=1, Hq=4, Hk=2, T=16, d=128, depth_alloc=3, depth_count=2, causal=1, scale=0.0, dtype=1)
    p, bad = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1008)

    def append(shape, slot, a=p):
        return L.moda_depth_append(a, p, p, p, slot, ctypes.byref(shape), None)

    assert append(MODAShape(**ok), 3) == 2                 # slot >= depth_alloc
    assert append(MODAShape(**ok), -1) == 2
    assert append(MODAShape(**ok), 0, a=None) == 1
    assert append(MODAShape(**ok), 0, a=bad) == 4
    assert append(MODAShape(**dict(ok, T=0)), 0) == 0      # empty: nothing launched
    assert append(MODAShape(**dict(ok, depth_alloc=0, depth_count=0)), 0) == 2

    def decode(shape, kv_alloc, ws=p, ws_bytes=1 << 30, q=p):
        return L.moda_attn_decode(q, p, p, p, p, p, p, kv_alloc, ws, ws_bytes, ctypes.byref(shape), None)

    need = L.moda_attn_decode_workspace_bytes(ctypes.byref(MODAShape(**ok)))
    assert need > 0
    assert decode(MODAShape(**ok), 15) == 2                # cache shorter than the attended length
    assert decode(MODAShape(**dict(ok, T=0)), 16) == 2     # the new token's own key is always attended
    assert decode(MODAShape(**dict(ok, dtype=0)), 16) == 3  # bf16 only
    assert decode(MODAShape(**ok), 16, ws=None) == 6
    assert decode(MODAShape(**ok), 16, ws_bytes=need - 1) == 6
    assert decode(MODAShape(**ok), 16, q=None) == 1
    assert decode(MODAShape(**ok), 16, q=bad) == 4
    assert decode(MODAShape(**dict(ok, B=0)), 16) == 0

    def bwd(shape, ws_bytes=1 << 30):
        return L.moda_attn_bwd(*([p] * 14), ws_bytes, ctypes.byref(shape), None)

    assert bwd(MODAShape(**dict(ok, Hq=256, Hk=2))) == 3   # more than 64 query heads per key/value head
    assert bwd(MODAShape(**dict(ok, dtype=0))) == 3
    assert bwd(MODAShape(**ok), ws_bytes=8) == 6
    assert L.moda_kernels_per_call(ctypes.byref(MODAShape(**ok)), 1) == 3               # up to 4 heads per group: the depth-slot gradients run inside dK/dV
    assert L.moda_kernels_per_call(ctypes.byref(MODAShape(**dict(ok, Hq=16))), 1) == 4  # 8 heads per group: a kernel of their own
    assert L.moda_kernels_per_call(ctypes.byref(MODAShape(**dict(ok, Hq=40))), 1) == 4  # 20 heads per group: likewise
    assert L.moda_kernels_per_call(ctypes.byref(MODAShape(**dict(ok, Hq=2))), 1) == 3
    assert L.moda_kernels_per_call(ctypes.byref(MODAShape(**ok)), 0) == 1


def test_size_limits_without_gpu(L):
    """One (batch, head) slab of a SEQUENCE tensor must stay below 4 GiB (32-bit byte offsets
    inside a slab); the depth tensors have no such limit (64-bit tile bases), only a cap on the
    slots per position; the decoding step addresses its caches with 64-bit pointers."""
    from paper_2603_15619_amd.binding import MODAFwdTuning, MODAShape

    p = ctypes.c_void_p(0x1000)
    base = dict(B=1, Hq=1, Hk=1, d=128, depth_count=1, causal=1, scale=0.0, dtype=1)

    def fwd_status(T, depth_alloc):
        s = MODAShape(T=T, depth_alloc=depth_alloc, **base)
        # NULL output pointer: a shape that passes validation stops at the pointer check
        return L.moda_attn_fwd(p, p, p, p, p, None, p, ctypes.byref(s), None)

    assert fwd_status(65536, 256) == 1          # 4 GiB of depth slots per head: accepted (then NULL output)
    assert fwd_status(131072, 8192) == 1
    assert fwd_status(65536, 8193) == 3         # more slots per position than the cap
    assert fwd_status((1 << 24) - 1, 1) == 1    # T * 128 * 2 bytes just below 4 GiB
    assert fwd_status(1 << 24, 1) == 3          # exactly 4 GiB: unsupported

    s = MODAShape(T=1 << 20, depth_alloc=256, **base)
    assert L.moda_attn_decode(p, p, p, p, p, None, p, 1 << 25, p, 1 << 30, ctypes.byref(s), None) == 1

    ok = MODAShape(B=1, Hq=4, Hk=2, T=16, d=128, depth_alloc=0, depth_count=0, causal=1, scale=0.0, dtype=1)

    def tuned(**kw):
        return L.moda_attn_fwd_tuned(p, p, p, None, None, None, p, ctypes.byref(ok), ctypes.byref(MODAFwdTuning(**kw)),
                                     None)

    assert tuned(waves=8, heads_per_tile=2, head_group=1) == 1   # accepted (then NULL output)
    assert tuned(waves=5) == 2 and tuned(heads_per_tile=4) == 2 and tuned(head_group=-2) == 2


def test_grids_of_2_to_the_32_threads_are_refused(L):
    """Before anything is launched (the runtime itself takes some of them and runs a part of the workgroups).  A backward
    call whose key and query tiles are too many for one launch keeps them apart."""
    from paper_2603_15619_amd.binding import MODAShape

    p = ctypes.c_void_p(0x1000)

    def shape(B, H, T, dtype=1):
        return ctypes.byref(MODAShape(B, H, H, T, 64, 0, 0, 1, 0.0, dtype))

    for T, B, dtype in ((1, 1 << 21, 1), (9, 1 << 21, 0), (128, 1 << 21, 1)):
        assert L.moda_attn_fwd(p, p, p, None, None, p, p, shape(B, 8, T, dtype), None) == 3
    assert L.moda_attn_decode(p, p, p, None, None, p, p, 1, p, 1 << 50, shape(1 << 21, 8, 1), None) == 3
    assert L.moda_attn_bwd(*([p] * 14), 1 << 50, shape(1 << 21, 8, 1), None) == 3
    for heads, kernels in ((1 << 22, 2), (1 << 23, 3)):
        assert L.moda_kernels_per_call(shape(heads // 8, 8, 17), 1) == kernels


@pytest.mark.parametrize("d,kernels", [(64, 3), (128, 4)])
def test_depth_gradients_of_5_to_8_heads_take_their_own_kernel_at_d_128(d, kernels):
    """Many key tiles, full blocks of slots: inside dK/dV at d = 64 only (at d = 128 the registers do not
    suffice and it would reload them from scratch memory at every position)."""
    from paper_2603_15619_amd.binding import MODAShape, lib

    for G in (5, 8):
        s = MODAShape(8, 8 * G, 8, 4096, d, 64, 64, 1, 0.0, 1)
        assert lib().moda_kernels_per_call(ctypes.byref(s), 1) == kernels


@pytest.mark.parametrize("B,Hq,Hk,d", [(8, 64, 8, 64), (8, 64, 8, 128), (4, 64, 8, 128), (2, 32, 4, 128), (1, 16, 16, 128),
                                       (3, 4, 2, 64), (600, 8, 1, 64), (64, 256, 4, 64), (5000, 8, 8, 64)])
def test_decode_workspace_of_the_longest_context_serves_shorter_ones(L, B, Hq, Hk, d):
    """The size never falls as the context grows."""
    from paper_2603_15619_amd.binding import MODAShape

    last = 0
    for T in [*range(1, 10000, 3), *range(10000, 70000, 61)]:
        n = L.moda_attn_decode_workspace_bytes(ctypes.byref(MODAShape(B, Hq, Hk, T, d, 4, 4, 1, 0.0, 1)))
        assert n >= last, (T, n, last)
        last = n


@pytest.mark.parametrize("T,B,kernels", [(1024, 4, 4), (512, 8, 4), (512, 20, 3), (1024, 9, 3), (1024, 8, 4)])
def test_few_key_tiles(L, T, B, kernels):
    """Few workgroups of 32 keys (2048 at most, fewer for short walks) take the dK/dV kernel that does without
    the depth slots of 8 heads: one kernel more."""
    from paper_2603_15619_amd.binding import MODAShape

    s = MODAShape(B, 64, 8, T, 64, 64, 64, 1, 0.0, 1)
    assert L.moda_kernels_per_call(ctypes.byref(s), 1) == kernels


@pytest.mark.parametrize("L_slots,kernels", [(21, 4), (22, 3), (32, 3), (33, 4), (43, 4), (44, 3), (64, 3), (0, 4)])
def test_depth_gradients_of_8_heads_inside_dkdv_where_blocks_of_32_slots_are_filled(L, L_slots, kernels):
    from paper_2603_15619_amd.binding import MODAShape

    s = MODAShape(8, 64, 8, 4096, 64, 64, L_slots, 1, 0.0, 1)
    assert L.moda_kernels_per_call(ctypes.byref(s), 1) == kernels


@pytest.mark.parametrize("B,Hq,Hk,T,d,slots,causal,dtype,tuned,name", [
    (1, 16, 16, 65536, 128, 15, 1, 1, None, "moda_fwd_bf16_kernel<128, 8, 2>"),
    (8, 16, 16, 513, 128, 1, 1, 1, None, "moda_fwd_bf16_kernel<128, 4, 2>"),   # one and a half rounds, up to 1024 positions
    (7, 12, 12, 1030, 128, 1, 1, 1, None, "moda_fwd_bf16_kernel<128, 8, 2>"),  # ... and more
    (29, 4, 4, 1000, 128, 0, 1, 1, None, "moda_fwd_bf16_kernel<128, 8, 2>"),   # more than one and three quarters
    (40, 13, 13, 240, 128, 12, 1, 1, None, "moda_fwd_bf16_kernel<128, 8, 2>"),  # many slots, little padding, two rounds
    (40, 13, 13, 230, 128, 12, 1, 1, None, "moda_fwd_bf16_kernel<128, 4, 2>"),
    (40, 13, 13, 240, 128, 11, 1, 1, None, "moda_fwd_bf16_kernel<128, 4, 2>"),
    (39, 13, 13, 240, 128, 12, 1, 1, None, "moda_fwd_bf16_kernel<128, 4, 2>"),
    (16, 16, 16, 240, 128, 12, 1, 1, None, "moda_fwd_bf16_kernel<128, 8, 2>"),  # ... or just one round
    (16, 17, 17, 240, 128, 12, 1, 1, None, "moda_fwd_bf16_kernel<128, 4, 2>"),
    (13, 12, 12, 1000, 64, 0, 1, 1, None, "moda_fwd_bf16_kernel<64, 4, 4>"),
    (13, 12, 12, 1030, 64, 0, 1, 1, None, "moda_fwd_bf16_kernel<64, 8, 4>"),
    (2, 16, 16, 1500, 64, 7, 1, 1, None, "moda_fwd_bf16_kernel<64, 4, 2>"),
    (2, 16, 16, 1500, 64, 7, 1, 1, dict(waves=8), "moda_fwd_bf16_kernel<64, 8, 4>"),
    (1, 12, 12, 2000, 64, 0, 0, 1, None, "moda_fwd_short_kernel<64, false>"),
    (1, 13, 13, 2000, 64, 0, 0, 1, None, "moda_fwd_bf16_kernel<64, 4, 2>"),
    (1, 2, 2, 100, 128, 3, 1, 1, None, "moda_fwd_short_kernel<128, true>"),
    (1, 2, 2, 100, 128, 3, 1, 1, dict(), "moda_fwd_bf16_kernel<128, 4, 2>"),
    (1, 2, 2, 256, 64, 4, 1, 0, None, "moda_fwd_f32_kernel<64>"),
    (1, 2, 2, 5, 64, 4, 1, 0, None, "moda_fwd_f32_rows_kernel<64>"),
    (0, 2, 2, 5, 64, 4, 1, 0, None, ""), (1, 2, 2, 5, 96, 4, 1, 1, None, ""), (1, 2, 2, 5, 64, 4, 1, 1, dict(waves=5), "")])
def test_forward_kernel_names(L, B, Hq, Hk, T, d, slots, causal, dtype, tuned, name):
    from paper_2603_15619_amd.binding import MODAFwdTuning, MODAShape

    s = MODAShape(B, Hq, Hk, T, d, slots, slots, causal, 0.0, dtype)
    tuning = None if tuned is None else ctypes.byref(MODAFwdTuning(**tuned))
    out = ctypes.create_string_buffer(64)
    assert L.moda_fwd_kernel_name(ctypes.byref(s), tuning, out, len(out)) == len(name)
    assert out.value.decode() == name
    cut = ctypes.create_string_buffer(8)
    L.moda_fwd_kernel_name(ctypes.byref(s), tuning, cut, len(cut))
    assert cut.value.decode() == name[:7]


@pytest.mark.parametrize("B,Hq,Hk,T,d,slots,causal,names", [
    (8, 16, 16, 4096, 128, 15, 1, ["moda_bwd_grads_kernel<128, 1, false, false, 4>"]),
    (2, 16, 8, 1000, 64, 12, 1, ["moda_bwd_grads_kernel<64, 2, true, true, 4>"]),
    # calls that a chain or a second round of 128-row tiles made slower than two launches, or than another kind
    (17, 8, 8, 192, 128, 64, 1, ["moda_bwd_grads_kernel<128, 1, true, true, 4>"]),
    (7, 8, 8, 537, 64, 64, 1, ["moda_bwd_grads_kernel<64, 1, true, true, 4>"]),
    (17, 8, 8, 264, 128, 31, 1, ["moda_bwd_grads_kernel<128, 1, true, true, 4>"]),
    (1, 8, 2, 5166, 64, 0, 1, ["moda_bwd_grads_kernel<64, 0, true, true, 8>"]),
    (3, 8, 1, 10305, 128, 0, 1, ["moda_bwd_grads_kernel<128, 0, true, false, 8>"]),
    (3, 4, 1, 13537, 128, 7, 1, ["moda_bwd_grads_kernel<128, 4, true, false, 8>"]),
    (1, 64, 8, 16384, 64, 64, 1, ["moda_bwd_dkdv_kernel<64, 8>", "moda_bwd_dq_kernel<64, 4, 2>"]),
    (1, 9, 1, 97, 128, 2, 1, ["moda_bwd_dkdv_short_kernel<128, 0, 4>", "moda_bwd_dq_short_kernel<128>"]),
    (1, 2, 2, 16, 64, 2, 1, ["moda_bwd_dkdv_short_kernel<64, 1, 4>", "moda_bwd_dq_short_kernel<64>"]),
    (0, 2, 2, 16, 64, 2, 1, [""]), (1, 65, 1, 16, 64, 2, 1, [""])])
def test_backward_kernel_names(L, B, Hq, Hk, T, d, slots, causal, names):
    from paper_2603_15619_amd.binding import MODAShape

    s = MODAShape(B, Hq, Hk, T, d, slots, slots, causal, 0.0, 1)
    for which in (0, 1):
        name = names[which % len(names)]
        out = ctypes.create_string_buffer(64)
        assert L.moda_bwd_kernel_name(ctypes.byref(s), which, out, len(out)) == len(name)
        assert out.value.decode() == name
    assert L.moda_bwd_kernel_name(ctypes.byref(s), 2, out, len(out)) == 0 and out.value == b""
