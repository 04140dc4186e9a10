"""The work that a program built on this framework has it do, as measurable cases.

Every case is one call, or for training one forward and backward pass, of a public entry point
of paper_2603_15619_amd:

  op "fwd"    moda_attn_fwd                 a layer's attention: prefill, evaluation
  op "bwd"    moda_attn_bwd                 its gradients, from a forward pass that is in hand
  op "train"  moda_attn_fwd, moda_attn_bwd  one layer of a training step
  op "decode" moda_attn_decode              one new token per sequence
  op "append" moda_depth_append             the depth stream's write step

with B sequences, Hq query heads on Hk key/value heads, T positions, head dimension d, L attended
depth slots of La allocated ones, kv_alloc rows in a decoding cache, and dtype "bf16" or "f32".
"""
import math

import torch

from paper_2603_15619_amd import (MODAShape, moda_attn_bwd, moda_attn_bwd_workspace_bytes, moda_attn_decode,
                                  moda_attn_fwd, moda_depth_append, synth)


def _case(op, B, Hq, Hk, T, d, L, La=None, dtype="bf16", causal=True, kv_alloc=None, name=None):
    c = {"op": op, "B": B, "Hq": Hq, "Hk": Hk, "T": T, "d": d, "L": L, "La": L if La is None else La,
         "dtype": dtype, "causal": causal, "kv_alloc": T if kv_alloc is None else kv_alloc}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the accuracy configuration: one small fp32 call, where launch and latency are what counts
        _case("fwd", 1, 2, 2, 256, 64, 4, dtype="f32", name="fwd_f32_tiny"),
        # a whole layer in fp32 at a length that no tile divides: a model checked in full precision
        _case("fwd", 1, 16, 16, 2000, 128, 15, dtype="f32", name="fwd_f32_layer"),
        # the deepest layer of a 16-layer 1.5B-parameter model on a batch of 4K sequences
        _case("fwd", 8, 16, 16, 4096, 128, 15, name="fwd_layer_4k"),
        # the same layer over one 64K context: the largest call
        _case("fwd", 1, 16, 16, 65536, 128, 15, name="fwd_long_64k"),
        # a middle layer (7 of 16 slots filled so far) on short ragged prompts
        _case("fwd", 2, 16, 16, 1000, 128, 7, La=16, name="fwd_short_ragged"),
        # a training step of a grouped-query layer at the paper's kernel-benchmark shape
        _case("train", 1, 64, 8, 16384, 64, 64, name="train_group_16k"),
        # a training step on short ragged sequences, two heads per group, half the slots filled
        _case("train", 2, 16, 8, 1000, 64, 12, La=24, name="train_short_ragged"),
        # the backward pass of the 1.5B-parameter model's deepest layer
        _case("bwd", 8, 16, 16, 4096, 128, 15, name="bwd_layer_4k"),
        # serving: a batch of 8 long contexts, one head per key/value head
        _case("decode", 8, 16, 16, 65536, 128, 15, name="decode_long_64k"),
        # serving: a single short chat, the smallest bf16 call
        _case("decode", 1, 16, 16, 1003, 128, 15, La=16, kv_alloc=2048, name="decode_short"),
        # serving with grouped queries (the paper's kernel geometry)
        _case("decode", 8, 64, 8, 65536, 64, 64, name="decode_group_64k"),
        # a layer's keys and values written to the depth cache of a 16-layer stack
        _case("append", 8, 16, 16, 4096, 128, 8, La=16, name="append_layer_4k"),
    ]


def _pairs(c):
    T = c["T"]
    seq = T * (T + 1) // 2 if c["causal"] else T * T
    return c["B"] * c["Hq"] * (seq + T * c["L"])


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: lengths over their logarithm, odd ones included; slots from none to 64, some
    allocated but not filled; one to eight heads per group; at most the largest listed case's work."""
    op = rng.choice(["fwd", "fwd", "fwd_f32", "train", "train", "bwd", "decode", "decode", "append"])
    d = rng.choice([64, 128])
    L = rng.choice([0, 1, 4, 7, 12, 15, 24, 31, 64])
    La = L + rng.choice([0, 0, 1, 5])
    G = rng.choice([1, 1, 2, 4, 8])
    Hk = rng.choice([2, 4, 8, 16]) if G <= 2 else rng.choice([1, 2, 4, 8])
    causal = rng.random() < 0.85
    if op == "decode":
        T = _log_int(rng, 64, 65536)
        B = min(_log_int(rng, 1, 32), max(1, (1 << 23) // (Hk * T)))
        return _case("decode", B, G * Hk, Hk, T, d, L, La, kv_alloc=T + rng.choice([0, 1, 64, 1000]))
    if op == "append":
        T = _log_int(rng, 64, 16384)
        B = min(_log_int(rng, 1, 8), max(1, (1 << 19) // (Hk * T)))
        La = max(La, 1)
        return _case("append", B, Hk, Hk, T, d, min(L, La - 1), La, dtype=rng.choice(["bf16", "bf16", "f32"]))
    if op == "fwd_f32":
        T = _log_int(rng, 64, 2048)
        return _case("fwd", rng.choice([1, 2]), G * min(Hk, 8 // G if G < 8 else 1), min(Hk, 8 // G if G < 8 else 1), T, d,
                     min(L, 31), min(La, 32), dtype="f32", causal=causal)
    T = _log_int(rng, 64, 16384)
    causal = causal or T > 8192  # (twice the pairs)
    B = min(_log_int(rng, 1, 8), max(1, (1 << 18) // (G * Hk * T)))
    return _case(op, B, G * Hk, Hk, T, d, L, La, causal=causal)


# ------------------------------------------------------------------------------------------ one pass
def prepare(case, seed):
    c = case
    if c["op"] == "decode":
        # the sequence cache (kv_alloc rows, T of them filled), the new token's queries and depth
        # slots, and the output and workspace buffers that a serving loop keeps
        seq = synth.make_inputs(c["B"], c["Hq"], c["Hk"], c["kv_alloc"], c["d"], 0, seed=2 * seed, device="cuda")
        one = synth.make_inputs(c["B"], c["Hq"], c["Hk"], 1, c["d"], c["L"], seed=2 * seed + 1, device="cuda",
                                depth_alloc=c["La"])
        st = {"Q": one["Q"][:, :, 0].contiguous(), "Kseq": seq["Kseq"], "Vseq": seq["Vseq"],
              "Kdepth": None if c["La"] == 0 else one["Kdepth"][:, :, 0].contiguous(),
              "Vdepth": None if c["La"] == 0 else one["Vdepth"][:, :, 0].contiguous()}
        st["out"] = torch.empty_like(st["Q"])
        st["lse"] = torch.empty((c["B"], c["Hq"]), dtype=torch.float32, device="cuda")
        st["workspace"] = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    elif c["op"] == "append":
        st = synth.make_inputs(c["B"], c["Hk"], c["Hk"], c["T"], c["d"], 0, dtype=c["dtype"], seed=seed, device="cuda",
                               depth_alloc=c["La"])
    else:
        st = synth.make_inputs(c["B"], c["Hq"], c["Hk"], c["T"], c["d"], c["L"], dtype=c["dtype"], seed=seed,
                               device="cuda", depth_alloc=c["La"], with_dO=c["op"] != "fwd")
        if c["op"] != "fwd":
            shape = MODAShape(c["B"], c["Hq"], c["Hk"], c["T"], c["d"], c["La"], c["L"], int(c["causal"]), 0.0, 1)
            st["workspace"] = torch.empty(moda_attn_bwd_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
        if c["op"] == "bwd":
            st["O"], st["LSE"] = moda_attn_fwd(st["Q"], st["Kseq"], st["Vseq"], st["Kdepth"], st["Vdepth"],
                                               depth_count=c["L"], causal=c["causal"])
    st["case"] = dict(c)
    return st


def run(state):
    c, s = state["case"], state
    if c["op"] == "decode":
        O, LSE = moda_attn_decode(s["Q"], s["Kseq"], s["Vseq"], s["Kdepth"], s["Vdepth"], T=c["T"], depth_count=c["L"],
                                  out=s["out"], lse=s["lse"], workspace=s["workspace"])
        return {"O": O, "LSE": LSE}
    if c["op"] == "append":
        Kd, Vd = moda_depth_append(s["Kseq"], s["Vseq"], s["Kdepth"], s["Vdepth"], c["L"])
        return {"Kdepth": Kd, "Vdepth": Vd}
    out = {}
    if c["op"] == "bwd":
        O, LSE = s["O"], s["LSE"]
    else:
        O, LSE = moda_attn_fwd(s["Q"], s["Kseq"], s["Vseq"], s["Kdepth"], s["Vdepth"], depth_count=c["L"],
                               causal=c["causal"])
        out = {"O": O, "LSE": LSE}
    if c["op"] != "fwd":
        grads = moda_attn_bwd(s["Q"], s["Kseq"], s["Vseq"], s["Kdepth"], s["Vdepth"], O, LSE, s["dO"],
                              depth_count=c["L"], causal=c["causal"], workspace=s["workspace"])
        out.update({k: g for k, g in zip(("dQ", "dKseq", "dVseq", "dKdepth", "dVdepth"), grads) if g is not None})
    return out


# ------------------------------------------------------------------------------------------ what it cannot do without
def work(case):
    """Bytes: every input that takes part read once, every output written once.  Operations: 4 d per
    visible (query, key) pair forward (two products), 10 d backward (five products)."""
    c = case
    B, Hq, Hk, T, d, L, La = (c[k] for k in ("B", "Hq", "Hk", "T", "d", "L", "La"))
    e = 2 if c["dtype"] == "bf16" else 4
    if c["op"] == "decode":
        return {"bytes": 2 * e * B * Hk * (T + L) * d + 2 * e * B * Hq * d + 4 * B * Hq,
                "flops": 4 * d * B * Hq * (T + L)}
    if c["op"] == "append":
        return {"bytes": 4 * e * B * Hk * T * d, "flops": 0}
    q, kv, dep, stat = e * B * Hq * T * d, e * B * Hk * T * d, e * B * Hk * T * d, 4 * B * Hq * T
    read = q + 2 * kv + 2 * L * dep            # Q, K, V and the attended slots
    grads = q + 2 * kv + 2 * La * dep          # dQ, dK, dV and every allocated slot's gradient
    if c["op"] == "fwd":
        return {"bytes": read + q + stat, "flops": 4 * d * _pairs(c)}
    if c["op"] == "bwd":
        return {"bytes": read + 2 * q + stat + grads, "flops": 10 * d * _pairs(c)}
    return {"bytes": read + 2 * q + stat + grads, "flops": 14 * d * _pairs(c)}  # reads dO, writes O, LSE and gradients


def tolerance(case):
    """Relative error of the worst output: four times what the path was seen to be off its 64-bit
    value.  fp32: 5e-7.  bf16 (weights, logit gradients and results rounded to 8 bits): 1.6e-3 to
    2.4e-3, forward and backward.  `max` is against an output's root mean square: single elements
    of a gradient can be the difference of much larger terms."""
    if case["op"] == "append":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 8e-5}
    return {"rel": 1e-2, "max": 0.4}


# ------------------------------------------------------------------------------------------ the same in 64 bits
def _attend(q, k, v, kd, vd, causal, row0, scale):
    """One (batch, head), some rows of queries (row0 ...): weights over sequence keys and over the
    rows' own slots, the output and the log-sum-exp."""
    s = (q @ k.t().contiguous()) * scale
    if causal:
        rows = torch.arange(row0, row0 + q.shape[0], device=q.device)
        s.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > rows[:, None], -math.inf)
    sd = (kd * q[:, None, :]).sum(-1) * scale
    lse = torch.logsumexp(torch.cat([s, sd], 1), 1)
    p, pd = torch.exp(s - lse[:, None]), torch.exp(sd - lse[:, None])
    return p, pd, p @ v + (pd[:, :, None] * vd).sum(1), lse


def exact(case, seed):
    c = case
    if c["op"] == "append":
        return None  # bytes are moved, nothing is computed
    B, Hq, Hk, T, d, L, La = (c[k] for k in ("B", "Hq", "Hk", "T", "d", "L", "La"))
    st = prepare(dict(c, op="train") if c["op"] == "bwd" else c, seed)
    G, scale, f64 = Hq // Hk, 1.0 / math.sqrt(d), dict(dtype=torch.float64, device="cuda")
    if c["op"] == "decode":
        O, LSE = torch.empty((B, Hq, d), **f64), torch.empty((B, Hq), **f64)
        none = torch.empty((1, 0, d), **f64)
        for b in range(B):
            for h in range(Hq):
                k, v = (st[n][b, h // G, :T].double() for n in ("Kseq", "Vseq"))
                kd, vd = (none if L == 0 else st[n][b, h // G, None, :L].double() for n in ("Kdepth", "Vdepth"))
                _, _, o, lse = _attend(st["Q"][b, h, None].double(), k, v, kd, vd, False, 0, scale)
                O[b, h], LSE[b, h] = o[0], lse[0]
        return {"O": O, "LSE": LSE}
    back = c["op"] != "fwd"
    out = {}
    if c["op"] != "bwd":
        out.update(O=torch.empty((B, Hq, T, d), **f64), LSE=torch.empty((B, Hq, T), **f64))
    if back:
        out.update(dQ=torch.empty((B, Hq, T, d), **f64), dKseq=torch.zeros((B, Hk, T, d), **f64),
                   dVseq=torch.zeros((B, Hk, T, d), **f64))
        if La:
            out.update(dKdepth=torch.zeros((B, Hk, T, La, d), **f64), dVdepth=torch.zeros((B, Hk, T, La, d), **f64))
    for b in range(B):
        for h in range(Hq):
            g = h // G
            q, k, v = (st[n][b, i].double() for n, i in (("Q", h), ("Kseq", g), ("Vseq", g)))
            for r0 in range(0, T, 2048):
                r1 = min(T, r0 + 2048)
                n = r1 if c["causal"] else T  # keys that some row of the chunk sees
                kd, vd = (torch.empty((r1 - r0, 0, d), **f64) if L == 0 else st[x][b, g, r0:r1, :L].double()
                          for x in ("Kdepth", "Vdepth"))
                p, pd, o, lse = _attend(q[r0:r1], k[:n], v[:n], kd, vd, c["causal"], r0, scale)
                if "O" in out:
                    out["O"][b, h, r0:r1], out["LSE"][b, h, r0:r1] = o, lse
                if back:
                    do = st["dO"][b, h, r0:r1].double()
                    delta = (do * o).sum(1, keepdim=True)
                    e = p * (do @ v[:n].t().contiguous() - delta) * scale
                    ed = pd * ((vd * do[:, None, :]).sum(-1) - delta) * scale
                    out["dQ"][b, h, r0:r1] = e @ k[:n] + (ed[:, :, None] * kd).sum(1)
                    out["dKseq"][b, g, :n] += e.t().contiguous() @ q[r0:r1]
                    out["dVseq"][b, g, :n] += p.t().contiguous() @ do
                    if L:
                        out["dKdepth"][b, g, r0:r1, :L] += ed[:, :, None] * q[r0:r1, None, :]
                        out["dVdepth"][b, g, r0:r1, :L] += pd[:, :, None] * do[:, None, :]
    return out
