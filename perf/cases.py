"""The calls whose speed is measured: what a program that serves a model on this
library has it do, through the public entry points of paper_2511_18936_amd.

  step       SwanCache.step: one decode step of a batch (append one token per
             sequence, attend over the cache); the cache grows by one token a pass
  append     SwanCache.append: a prompt, or a chunk of one, into the cache
  change_k   swan.change_k: the caches of running sequences laid out for another k
  calibrate  swan.calibrate_rotation: one head's rotation from its rows
  joint      layer.calibrate_joint: both rotations of every kv head of a layer
  rope       swan.rope: query or key rows at their positions
  layer      SwanAttentionLayer: a prompt through a layer, then its first token

Cached rows follow the low-rank recipe of the repository's benchmark: rows =
Z . diag(s) . R with s_j = exp(-j / 16) and one random rotation R per head, and the
rotations that a calibration on such rows finds (R transposed).
"""
import math

import torch

from paper_2511_18936_amd import swan
from paper_2511_18936_amd.layer import SwanAttentionLayer, calibrate_joint

D = swan.HEAD_DIM
DEVICE = "cuda"
WINDOW = 512  # decode steps before a cache's lengths go back to where they began
FP16 = {"f16": torch.float16, "f32": torch.float32}


def listed():
    return [
        # one user, a short chat: a decode step where launches and latencies are the time
        dict(name="step_mha_4k_b1", kind="step", batch=1, q_heads=32, kv_heads=32, length=4095,
             buffer=128, k=64, k_value=0, mix="", dtype="f16", values="same", ragged=False),
        # a full serving batch at long context: a decode step bound by the cache's bytes
        dict(name="step_mha_32k_b16", kind="step", batch=16, q_heads=32, kv_heads=32,
             length=32767, buffer=128, k=48, k_value=0, mix="", dtype="f16", values="same",
             ragged=False),
        # grouped-query heads, a few very long documents
        dict(name="step_gqa_128k_b4", kind="step", batch=4, q_heads=32, kv_heads=8,
             length=131071, buffer=256, k=64, k_value=0, mix="", dtype="f16", values="same",
             ragged=False),
        # grouped-query heads and 8-bit values, a continuous batch of sequences at all lengths
        dict(name="step_gqa_ragged_e4m3", kind="step", batch=24, q_heads=32, kv_heads=8,
             length=32768, buffer=128, k=64, k_value=0, mix="", dtype="f16", values="e4m3",
             ragged=True),
        # k chosen per sequence by its user's memory budget
        dict(name="step_mha_mixed_k_16k_b8", kind="step", batch=8, q_heads=32, kv_heads=32,
             length=16384, buffer=128, k=0, k_value=0, mix="32,48,64,96", dtype="f16",
             values="same", ragged=False),
        # the prompts of a batch at once, k per sequence
        dict(name="prefill_mha_16k_b8", kind="append", batch=8, q_heads=32, kv_heads=32,
             cached=0, new=16384, buffer=128, k=0, k_value=0, mix="32,48,64,96", dtype="f16",
             values="same", ragged=False),
        # one user's prompt of ordinary length, the time to the first token
        dict(name="prefill_gqa_1k_b1", kind="append", batch=1, q_heads=32, kv_heads=8,
             cached=0, new=1009, buffer=128, k=64, k_value=0, mix="", dtype="f16",
             values="same", ragged=False),
        # a chunk of tokens for running sequences (chunked prompts, verified drafts)
        dict(name="append_40_gqa_b8", kind="append", batch=8, q_heads=32, kv_heads=8,
             cached=2000, new=40, buffer=128, k=64, k_value=0, mix="", dtype="f16",
             values="same", ragged=False),
        # float32 storage, as a model is checked before it is put to 16 bits
        dict(name="prefill_f32_2k_b2", kind="append", batch=2, q_heads=32, kv_heads=32,
             cached=0, new=2047, buffer=64, k=64, k_value=0, mix="", dtype="f32",
             values="same", ragged=False),
        # a layer's rotations from its activations and weights, offline
        dict(name="calibrate_joint_gqa", kind="joint", q_heads=32, kv_heads=8, tokens=1024,
             hidden=4096),
        # memory taken back from running sequences
        dict(name="change_k_64_to_40_16k_b4", kind="change_k", batch=4, kv_heads=32,
             length=16384, buffer=128, k=64, k_to=40, dtype="f16", values="same"),
        # a whole attention layer: prompt, then the first generated token
        dict(name="layer_prompt_gqa_2k", kind="layer", batch=1, q_heads=32, kv_heads=8,
             hidden=4096, new=1999, buffer=128, k=64, dtype="f16", values="same"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    return rng.choice([(32, 32), (32, 8), (32, 8), (8, 8), (24, 8), (16, 2), (16, 1)])


def _format(rng):
    r = rng.random()
    return ("f32", "same") if r < 0.15 else ("f16", "e4m3") if r < 0.5 else ("f16", "same")


def _ks(rng):
    """(k, k_value, mix): one k, keys and values with their own, or k per sequence."""
    r = rng.random()
    if r < 0.2:
        return 0, 0, "32,48,64,96"
    k = rng.randint(16, 96)
    return k, (rng.randint(16, 96) if r < 0.4 else 0), ""


def draw(rng):
    kind = rng.choice(["step", "step", "step", "append", "append", "change_k", "calibrate",
                       "joint", "rope", "layer"])
    dtype, values = _format(rng)
    if kind == "step":
        hq, hkv = _heads(rng)
        batch = _log_int(rng, 1, 32)
        k, kv, mix = _ks(rng)
        most = 16 * 32 * 32768 * 48 * 3 / (batch * hkv * 96 * (5 if dtype == "f32" else 3))
        return dict(kind=kind, batch=batch, q_heads=hq, kv_heads=hkv,
                    length=_log_int(rng, 100, int(min(131072, most))),
                    buffer=rng.choice([16, 64, 128, 256]), k=k, k_value=kv, mix=mix, dtype=dtype,
                    values=values, ragged=batch > 1 and rng.random() < 0.5)
    if kind == "append":
        hq, hkv = _heads(rng)
        batch = _log_int(rng, 1, 16)
        k, kv, mix = _ks(rng)
        most = 8 * 32 * 16384 / (batch * hkv * (8 if dtype == "f32" else 1))
        new = _log_int(rng, 2, int(min(32768, most)))
        return dict(kind=kind, batch=batch, q_heads=hq, kv_heads=hkv,
                    cached=rng.choice([0, 0, rng.randint(1, 3000)]), new=new,
                    buffer=rng.choice([16, 64, 128, 256]), k=k, k_value=kv, mix=mix, dtype=dtype,
                    values=values, ragged=batch > 1 and rng.random() < 0.3)
    if kind == "change_k":
        hkv = rng.choice([8, 32])
        batch = _log_int(rng, 1, 16)
        k = rng.randint(24, 96)
        k_to = rng.choice([rng.randint(16, max(16, k - 1)), rng.randint(k, 104)])
        return dict(kind=kind, batch=batch, kv_heads=hkv,
                    length=_log_int(rng, 300, int(16 * 32 * 8192 / (batch * hkv))), buffer=128,
                    k=k, k_to=k_to, dtype=dtype, values=values)
    if kind == "calibrate":
        return dict(kind=kind, rows=_log_int(rng, 256, 65536))
    if kind == "joint":
        hq, hkv = rng.choice([(32, 8), (8, 8), (24, 8), (16, 2)])
        return dict(kind=kind, q_heads=hq, kv_heads=hkv, tokens=_log_int(rng, 128, 2048),
                    hidden=128 * rng.randint(4, 32))
    if kind == "rope":
        heads = rng.choice([8, 32])
        return dict(kind=kind, batch=_log_int(rng, 1, 16), heads=heads, new=_log_int(rng, 1, 8192),
                    position=rng.randint(0, 100000), dtype=dtype)
    hq, hkv = rng.choice([(32, 32), (32, 8), (16, 8), (24, 8)])
    return dict(kind=kind, batch=_log_int(rng, 1, 4), q_heads=hq, kv_heads=hkv,
                hidden=hq * D, new=_log_int(rng, 100, 4096), buffer=rng.choice([64, 128, 256]),
                k=rng.randint(32, 96), dtype="f16", values=values)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed, what):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000003 * int(seed) + what)
    return g


def _rotations(seed, heads, what):
    """One random rotation per head, float64 on the host."""
    g = torch.Generator()
    g.manual_seed(7919 * int(seed) + what)
    q, r = torch.linalg.qr(torch.randn(heads, D, D, dtype=torch.float64, generator=g))
    return q * torch.sign(torch.diagonal(r, dim1=-2, dim2=-1)).unsqueeze(-2)


def _rows(seed, what, R, batch, n, dtype):
    """[batch][heads][n][D] rows of the recipe; R [heads][D][D]."""
    g = _generator(seed, what)
    s = torch.exp(-torch.arange(D, device=DEVICE, dtype=torch.float32) / 16)
    out = torch.empty(batch, R.shape[0], n, D, dtype=dtype, device=DEVICE)
    for h in range(R.shape[0]):
        M = s.unsqueeze(1) * R[h].to(DEVICE, torch.float32)
        z = torch.randn(batch, n, D, generator=g, device=DEVICE)
        out[:, h] = (z @ M).to(dtype)
    return out


def _lengths(case, longest):
    """Tokens per sequence: all the longest, or spread from a twentieth of it up to it."""
    if not case.get("ragged"):
        return [longest] * case["batch"]
    return [max(1, round(longest * (1.0 if b == 0 else 0.05 + 0.95 * ((0.618034 * b) % 1))))
            for b in range(case["batch"])]


def _k_lists(case):
    if case.get("mix"):
        several = [int(x) for x in case["mix"].split(",")]
        return [several[b % len(several)] for b in range(case["batch"])], None
    kv = case.get("k_value") or 0
    return [case["k"]] * case["batch"], ([kv] * case["batch"] if kv else None)


def _kv_inputs(case, seed, n):
    """Rotations and n raw key and value rows per sequence and head."""
    dtype = FP16[case["dtype"]]
    Rk, Rv = _rotations(seed, case["kv_heads"], 1), _rotations(seed, case["kv_heads"], 2)
    k = _rows(seed, 1, Rk, case["batch"], n, dtype)
    v = _rows(seed, 2, Rv, case["batch"], n, dtype)
    P = [R.transpose(1, 2).to(torch.float32).contiguous().to(DEVICE) for R in (Rk, Rv)]
    return k, v, P[0], P[1]


def _cache(case, longest):
    k, kv = _k_lists(case)
    return swan.SwanCache(case["batch"], case.get("q_heads", case["kv_heads"]),
                          case["kv_heads"], case["buffer"],
                          max(0, longest - case["buffer"]), k, FP16[case["dtype"]], DEVICE,
                          sparse_values=case["values"], k_value=kv)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        L = case["length"]
        k, v, Pk, Pv = _kv_inputs(case, seed, L + 1)
        cache = _cache(case, L + WINDOW)
        lengths = _lengths(case, L)
        cache.append(k[:, :, :L].contiguous(), v[:, :, :L].contiguous(), Pk, Pv,
                     n_new_per_seq=lengths)
        q = torch.randn(case["batch"], case["q_heads"], D, generator=_generator(seed, 3),
                        device=DEVICE).to(FP16[case["dtype"]])
        return dict(kind=kind, cache=cache, start=list(cache.seq_len), P_qk=Pk, P_vo=Pv, q=q,
                    k=k[:, :, L:].contiguous(), v=v[:, :, L:].contiguous())
    if kind == "append":
        n, old = case["new"], case["cached"]
        k, v, Pk, Pv = _kv_inputs(case, seed, old + n)
        cache = _cache(case, old + n)
        if old:
            cache.append(k[:, :, :old].contiguous(), v[:, :, :old].contiguous(), Pk, Pv)
        return dict(kind=kind, cache=cache, start=list(cache.seq_len), P_qk=Pk, P_vo=Pv,
                    k=k[:, :, old:].contiguous(), v=v[:, :, old:].contiguous(),
                    per_seq=_lengths(case, n) if case["ragged"] else None)
    if kind == "change_k":
        k, v, Pk, Pv = _kv_inputs(case, seed, case["length"])
        cache = _cache(case, case["length"])
        cache.append(k, v, Pk, Pv)
        to = swan.SwanCache(case["batch"], case["kv_heads"], case["kv_heads"], case["buffer"],
                            max(0, case["length"] - case["buffer"]),
                            [case["k_to"]] * case["batch"], FP16[case["dtype"]], DEVICE,
                            sparse_values=case["values"])
        to.k_ring, to.v_ring = cache.k_ring, cache.v_ring  # the dense buffer stays where it is
        to.desc.k_ring, to.desc.v_ring = cache.desc.k_ring, cache.desc.v_ring
        return dict(kind=kind, cache=cache, to=to)
    if kind == "calibrate":
        R = _rotations(seed, 1, 1)
        return dict(kind=kind, rows=_rows(seed, 1, R, 1, case["rows"], torch.float32)[0, 0],
                    P=torch.empty(D, D, device=DEVICE), sigma=torch.empty(D, device=DEVICE),
                    workspace=torch.empty(swan.calibrate_workspace_bytes(D), dtype=torch.uint8,
                                          device=DEVICE))
    if kind == "joint":
        hq, hkv, n = case["q_heads"], case["kv_heads"], case["tokens"]
        k = _rows(seed, 1, _rotations(seed, hkv, 1), 1, n, torch.float16)[0]
        v = _rows(seed, 2, _rotations(seed, hkv, 2), 1, n, torch.float16)[0]
        g = _generator(seed, 3)
        # the group's queries share their kv head's directions, as post-RoPE queries do
        Rq = _rotations(seed, hkv, 1).repeat_interleave(hq // hkv, dim=0)
        q = _rows(seed, 4, Rq, 1, n, torch.float16)[0]
        W_o = (torch.randn(hq * D, case["hidden"], generator=g, device=DEVICE)
               / math.sqrt(hq * D)).to(torch.float16)
        return dict(kind=kind, q=q, k=k, v=v, W_o=W_o, kv_heads=hkv,
                    P_qk=torch.empty(hkv, D, D, device=DEVICE),
                    P_vo=torch.empty(hkv, D, D, device=DEVICE))
    if kind == "rope":
        x = torch.randn(case["batch"], case["heads"], case["new"], D,
                        generator=_generator(seed, 1), device=DEVICE).to(FP16[case["dtype"]])
        return dict(kind=kind, x=x, y=torch.empty_like(x),
                    position=[case["position"] + 17 * b for b in range(case["batch"])])
    # layer
    hq, hkv, hidden = case["q_heads"], case["kv_heads"], case["hidden"]
    W, P = _layer_weights(case, seed)
    layer = SwanAttentionLayer(W["q"], W["k"], W["v"], W["o"], P[0], P[1], hq, hkv, 500000.0,
                               case["batch"], case["buffer"], case["new"] + 1 - case["buffer"]
                               if case["new"] + 1 > case["buffer"] else 0,
                               [case["k"]] * case["batch"], sparse_values=case["values"])
    x, x1 = _layer_inputs(case, seed)
    return dict(kind="layer", layer=layer, x=x, x1=x1)


def _layer_weights(case, seed):
    g = _generator(seed, 5)
    hq, hkv, hidden = case["q_heads"], case["kv_heads"], case["hidden"]

    def w(rows, cols):
        return (torch.randn(rows, cols, generator=g, device=DEVICE) / math.sqrt(rows)).to(
            torch.float16)

    W = dict(q=w(hidden, hq * D), k=w(hidden, hkv * D), v=w(hidden, hkv * D),
             o=w(hq * D, hidden))
    P = [_rotations(seed, hkv, w).transpose(1, 2).to(torch.float32).contiguous().to(DEVICE)
         for w in (1, 2)]
    # keys and values with the recipe's spectrum in the rotations' bases
    s = torch.exp(-torch.arange(D, device=DEVICE, dtype=torch.float32) / 16)
    for name, Pr in (("k", P[0]), ("v", P[1])):
        for h in range(hkv):
            block = W[name][:, h * D:(h + 1) * D].float()
            W[name][:, h * D:(h + 1) * D] = ((block * s) @ Pr[h].T).to(torch.float16)
    return W, P


def _layer_inputs(case, seed):
    g = _generator(seed, 6)
    x = torch.randn(case["batch"], case["new"] + 1, case["hidden"], generator=g, device=DEVICE)
    x = x.to(torch.float16)
    return x[:, :-1].contiguous(), x[:, -1:].contiguous()


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _arrays(cache):
    return {"k_pages": cache.k_pages, "v_pages": cache.v_pages, "k_ring": cache.k_ring,
            "v_ring": cache.v_ring}


def run(state):
    kind = state["kind"]
    if kind == "step":
        cache = state["cache"]
        if cache.seq_len[0] >= state["start"][0] + WINDOW:
            cache.seq_len = list(state["start"])
        out = cache.step(state["k"], state["v"], state["q"], state["P_qk"], state["P_vo"])
        return {"out": out, **_arrays(cache)}
    if kind == "append":
        cache = state["cache"]
        cache.seq_len = list(state["start"])
        cache.append(state["k"], state["v"], state["P_qk"], state["P_vo"],
                     n_new_per_seq=state["per_seq"])
        return _arrays(cache)
    if kind == "change_k":
        a, b = state["cache"], state["to"]
        swan.change_k(a.desc, a.k_active, a.k_value, b.desc, b.k_active, b.k_value, a.seq_len)
        return {"k_pages": b.k_pages, "v_pages": b.v_pages}
    if kind == "calibrate":
        swan.calibrate_rotation(state["rows"], state["P"], state["sigma"], state["workspace"])
        return {"P": state["P"], "sigma": state["sigma"]}
    if kind == "joint":
        calibrate_joint(state["q"], state["k"], state["v"], state["W_o"], state["kv_heads"],
                        state["P_qk"], state["P_vo"])
        return {"P_qk": state["P_qk"], "P_vo": state["P_vo"]}
    if kind == "rope":
        return swan.rope(state["x"], state["position"], 500000.0, out=state["y"])
    layer = state["layer"]
    layer.cache.seq_len = [0] * layer.cache.batch
    layer(state["x"])
    y = layer(state["x1"])
    return {"y": y, **_arrays(layer.cache)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _value_bytes(case):
    return 4 if case["dtype"] == "f32" else 1 if case["values"] == "e4m3" else 2


def _rotation_flops(vectors):
    return 2.0 * D * D * vectors


def work(case):
    kind = case["kind"]
    if kind == "calibrate":
        n = case["rows"]
        return {"bytes": 4.0 * D * n + 4 * D * (D + 1), "flops": float(n) * D * (D + 1) + 9.0 * D ** 3}
    if kind == "joint":
        hq, hkv, n, hidden = (case[x] for x in ("q_heads", "kv_heads", "tokens", "hidden"))
        rows = (hq + 2 * hkv) * n + hq * hidden  # of all the joint matrices
        return {"bytes": 2.0 * D * rows + 8.0 * hkv * D * D,
                "flops": float(rows) * D * (D + 1) + 2 * hkv * 9.0 * D ** 3}
    if kind == "rope":
        n = case["batch"] * case["heads"] * case["new"]
        e = 4 if case["dtype"] == "f32" else 2
        return {"bytes": 2.0 * n * D * e, "flops": 3.0 * n * D}
    e = 4 if case["dtype"] == "f32" else 2
    hkv, b, buf = case["kv_heads"], case["batch"], case["buffer"]
    entry = _value_bytes(case) + 1
    if kind == "change_k":
        tokens = b * hkv * max(0, case["length"] - buf)
        return {"bytes": 2.0 * tokens * (case["k"] + case["k_to"]) * entry, "flops": 0.0}
    hq = case["q_heads"]
    ks, kvs = _k_lists(case)
    kvs = kvs or ks
    P = 2.0 * hkv * D * D * 4
    if kind == "step":
        by, fl = P + b * D * e * (2.0 * hkv + 2.0 * hq), _rotation_flops(b * 2.0 * (hkv + hq))
        for L, k, kv in zip(_lengths(case, case["length"]), ks, kvs):
            L += 1
            S = max(0, L - buf)
            by += hkv * (S * (k + kv) * entry + 2.0 * D * e * min(L, buf))
            fl += hq * (2.0 * S * (k + kv) + 4.0 * D * min(L, buf))
        return {"bytes": by, "flops": fl}
    new = _lengths(case, case["new"])
    old = case.get("cached", 0)
    by, fl = P, 0.0
    for n, k, kv in zip(new, ks, kvs):
        out = min(old + n, old + n - buf) - max(0, old - buf)  # tokens that leave the buffer
        by += hkv * (2.0 * D * e * n + max(0, out) * (k + kv) * entry + 2.0 * D * e * min(n, buf))
        fl += _rotation_flops(2.0 * hkv * n)
    if kind == "append":
        return {"bytes": by, "flops": fl}
    # layer: the projections, the prompt's append, one token's step
    cols, hidden = (hq + 2 * hkv) * D, case["hidden"]
    rows = b * (case["new"] + 1)
    by += 2.0 * (hidden * cols + hq * D * hidden + rows * hidden + b * hidden)
    S = max(0, case["new"] + 1 - buf)
    by += b * hkv * (S * 2.0 * case["k"] * entry + 4.0 * D * min(case["new"] + 1, buf))
    fl += 2.0 * rows * hidden * cols + 2.0 * b * hq * D * hidden + b * hq * 4.0 * S * case["k"]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind in ("calibrate", "joint"):
        return {"rel": 2e-7, "max": 1e-5}   # float64 solves, rounded to float32
    if kind == "change_k":
        return "exact"                      # stored pairs are moved, not computed
    if kind == "append":
        # float16: the exact rotation rounded once.  float32: float64 sums, whose
        # order can move the rounding of one value in some 10^7
        return "exact" if case["dtype"] == "f16" else {"rel": 1.2e-7, "max": 1e-6, "differ": 1e-6}
    if kind == "rope":  # float64, rounded once
        return {"rel": 8e-4, "max": 2e-3} if case["dtype"] == "f16" else {"rel": 1.2e-7, "max": 1e-6}
    if kind == "step":  # float32 sums over the tokens, rounded once to the storage type
        if case["dtype"] == "f16":
            return {"rel": 8e-4, "max": 4e-3}
        return {"rel": 2e-6, "max": 4e-5, "differ": 1e-6}
    # float16 products in front of the pruning: a rounding there can exchange a
    # row's k-th and (k+1)-th components (0.0026 to 0.005 off the 64-bit layer)
    return {"rel": 1.2e-2, "max": 0.3, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _store(x, case):
    return x.to(FP16[case["dtype"]]).double()


def _pruned(xh, k, case):
    """The k largest magnitudes of each row (ties: lower index), the rest zero, the kept
    values as the sparse cache stores them."""
    a = xh.abs()
    tau = torch.sort(a, dim=-1, descending=True).values[..., k - 1:k]
    above, at = a > tau, a == tau
    keep = above | (at & (torch.cumsum(at, -1) <= k - above.sum(-1, keepdim=True)))
    x = torch.where(keep, xh, torch.zeros((), dtype=xh.dtype, device=xh.device))
    return x.to(torch.float8_e4m3fn).double() if case["values"] == "e4m3" else x


def _attend(q, kh, vh, k, kv, buf, case):
    """One kv head: q [G][D] rotated, kh and vh [L][D] stored; the weighted sum of values."""
    S = max(0, kh.shape[0] - buf)
    keys = torch.cat([_pruned(kh[:S], k, case), kh[S:]])
    vals = torch.cat([_pruned(vh[:S], kv, case), vh[S:]])
    return torch.softmax(q @ keys.T / math.sqrt(D), dim=-1) @ vals


def _ring(xh, buf):
    """The buffer's rows by slot, of one kv head's rotated rows."""
    L = xh.shape[0]
    ring = torch.zeros(buf, D, dtype=torch.float64, device=xh.device)
    at = torch.arange(max(0, L - buf), L, device=xh.device)
    ring[at % buf] = xh[at]
    return ring


def exact(case, seed):
    kind = case["kind"]
    if kind == "change_k":
        return None
    if kind == "rope":
        s = prepare(case, seed)
        x = s["x"].double()
        pos = torch.tensor(s["position"], dtype=torch.float64, device=DEVICE)[:, None] + \
            torch.arange(case["new"], dtype=torch.float64, device=DEVICE)
        freq = 500000.0 ** (-torch.arange(D // 2, dtype=torch.float64, device=DEVICE) * 2 / D)
        ang = (pos[..., None] * freq)[:, None]
        a, b = x[..., :D // 2], x[..., D // 2:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)
    if kind in ("calibrate", "joint"):
        s = prepare(case, seed)
        if kind == "calibrate":
            P, sigma = _singular(s["rows"])
            return {"P": P, "sigma": sigma}
        G = case["q_heads"] // case["kv_heads"]
        Pq, Pv = [], []
        for h in range(case["kv_heads"]):
            W = s["W_o"].view(case["q_heads"], D, case["hidden"])[h * G:(h + 1) * G]
            Pq.append(_singular(torch.cat([s["q"][h * G:(h + 1) * G].reshape(-1, D), s["k"][h]]))[0])
            Pv.append(_singular(torch.cat([s["v"][h], W.transpose(1, 2).reshape(-1, D)]))[0])
        return {"P_qk": torch.stack(Pq), "P_vo": torch.stack(Pv)}
    if kind == "layer":
        return _exact_layer(case, seed)
    n = case["length"] + 1 if kind == "step" else case["cached"] + case["new"]
    k, v, Pk, Pv = _kv_inputs(case, seed, n)
    ks, kvs = _k_lists(case)
    hkv, buf = case["kv_heads"], case["buffer"]
    kr = torch.zeros(case["batch"], hkv, buf, D, dtype=torch.float64, device=DEVICE)
    vr = torch.zeros_like(kr)
    out = None
    if kind == "step":
        G = case["q_heads"] // hkv
        q = torch.randn(case["batch"], case["q_heads"], D, generator=_generator(seed, 3),
                        device=DEVICE).to(FP16[case["dtype"]]).double()
        out = torch.empty_like(q)
        lengths = _lengths(case, case["length"])
    else:
        lengths = [case["cached"] + m for m in _lengths(case, case["new"])]
    for b in range(case["batch"]):
        L = lengths[b]
        for h in range(hkv):
            rows = [x[b, h, :L] for x in (k, v)]
            if kind == "step":  # the step's own token
                rows = [torch.cat([r, x[b, h, -1:]]) for r, x in zip(rows, (k, v))]
            kh, vh = rows[0].double() @ Pk[h].double(), rows[1].double() @ Pv[h].double()
            kr[b, h], vr[b, h] = _ring(kh, buf), _ring(vh, buf)
            if kind == "step":
                hs = slice(h * G, (h + 1) * G)
                o = _attend(q[b, hs] @ Pk[h].double(), _store(kh, case), _store(vh, case), ks[b],
                            (kvs or ks)[b], buf, case)
                out[b, hs] = o @ Pv[h].double().T
    rings = {"k_pages": None, "v_pages": None, "k_ring": kr, "v_ring": vr}
    return rings if out is None else {"out": out, **rings}


def _singular(rows):
    """Right singular vectors (largest entry of each positive) and singular values."""
    S = rows.double()
    lam, V = torch.linalg.eigh((S.T @ S).cpu())
    lam, V = lam.flip(0), V.flip(1)
    big = V.gather(0, V.abs().argmax(0, keepdim=True))
    return V * torch.sign(big), lam.clamp(min=0).sqrt()


def _exact_layer(case, seed):
    hq, hkv, buf, k = case["q_heads"], case["kv_heads"], case["buffer"], case["k"]
    G = hq // hkv
    W, P = _layer_weights(case, seed)
    x, x1 = _layer_inputs(case, seed)
    x = torch.cat([x, x1], dim=1).double()
    B, n, _ = x.shape
    freq = 500000.0 ** (-torch.arange(D // 2, dtype=torch.float64, device=DEVICE) * 2 / D)
    ang = torch.arange(n, dtype=torch.float64, device=DEVICE)[:, None] * freq

    def rope(z, a):
        p, r = z[..., :D // 2], z[..., D // 2:]
        return torch.cat([p * a.cos() - r * a.sin(), r * a.cos() + p * a.sin()], -1)

    y = torch.zeros(B, case["hidden"], dtype=torch.float64, device=DEVICE)
    kr = torch.zeros(B, hkv, buf, D, dtype=torch.float64, device=DEVICE)
    vr = torch.zeros_like(kr)
    for b in range(B):
        for h in range(hkv):
            kh = rope(x[b] @ W["k"][:, h * D:(h + 1) * D].double(), ang) @ P[0][h].double()
            vh = x[b] @ W["v"][:, h * D:(h + 1) * D].double() @ P[1][h].double()
            kr[b, h], vr[b, h] = _ring(kh, buf), _ring(vh, buf)
            hs = slice(h * G, (h + 1) * G)
            q = (x[b, -1] @ W["q"][:, h * G * D:(h + 1) * G * D].double()).view(G, D)
            o = _attend(rope(q, ang[-1]) @ P[0][h].double(), _store(kh, case), _store(vh, case),
                        k, k, buf, case) @ P[1][h].double().T
            y[b] += o.reshape(-1) @ W["o"].view(hq, D, -1)[hs].reshape(G * D, -1).double()
    return {"y": y, "k_pages": None, "v_pages": None, "k_ring": kr, "v_ring": vr}
