"""Compress-append of several tokens at once, bit-exact against the oracle: the prefill
kernel (long appends of a large batch) at the edges of its units of 32 positions, with
several units a wave, values given in the rotated basis and every fp16 value, and the
insert kernel (everything else) at the edges of its blocks, for every remainder of
k by 8, masks in one half of the dims, ties and extreme rows."""
import numpy as np
import pytest

import swan_inputs as si
from tests import swan_cases as C
from oracle import swan_oracle as O
from tests.test_append_plan_host import PREFILL, append_kernel
from tests.test_gpu_e4m3 import _finite_fp16_rows
from tests.test_gpu_parity import _build, _extreme_rows

pytestmark = pytest.mark.gpu

B = 64  # 256 units of (sequence, kv head, role), so that 3 blocks each go to the prefill kernel
EDGES = [1, 2, 7, 8, 9, 15, 31, 32, 33, 40, 48, 63, 64, 65, 77, 96, 102, 120, 121, 127, 128]


def _check(cache, oc, Ls, dtype_np=np.float16, values="same"):
    for bi, L in enumerate(Ls):
        for h in range(len(oc[bi])):
            C.compare_unit(cache, oc[bi][h], bi, h, L, dtype_np, values)


def _one_half(K, V):
    """Values of a few equal magnitudes (ties everywhere), in the low half of the dims,
    the high half, or every 8th dim, depending on the token."""
    for X in (K, V):
        for t in range(X.shape[2]):
            row = np.zeros(128)
            d = np.arange(128)
            on = (d < 64, d >= 64, d % 8 == t % 8, d % 2 == 0)[t % 4]
            row[on] = np.where(d[on] % 3 == 0, -0.5, 0.25)
            X[:, :, t] = row.astype(X.dtype)


@pytest.mark.parametrize("first,b,hook,values", [
    (0, 0, None, "same"), (0, 33, _extreme_rows, "same"), (37, 16, None, "same"),
    (64, 128, _extreme_rows, "same"), (37, 0, None, "e4m3"),
])
def test_prefill_units(gpu_device, swan_mod, torch_mod, first, b, hook, values):
    # the last append: 256 to 300 tokens for some sequences, as few as 1 or none for others
    Ls = [first + (0, 1, 31, 32, 33, 64, 95, 256, 257, 288, 299, 300)[i % 12] for i in range(B)]
    Ls = [max(L, 1) for L in Ls]
    Ls[0] = first + 300
    ks = [EDGES[i % len(EDGES)] for i in range(B)]
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=B, Hq=2, Hkv=2, L=Ls, b=b,
                           k_active=ks, dtype="f16", values=values, kv_hook=hook,
                           chunks=[first, 300] if first else [300])
    _check(cache, oc, Ls, values=values)


@pytest.mark.parametrize("heads", [2, 3, 5])
@pytest.mark.parametrize("old", [0, 37])
def test_prefill_short_chunks(gpu_device, swan_mod, torch_mod, old, heads):
    """Chunks of 160 to 191 tokens of every sequence, the shortest that go to it, of
    (head, role) pairs that are no multiple of the XCDs."""
    Ls = [old + 160 + (7 * i) % 32 for i in range(B)]
    Ls[0] = old + 191
    assert append_kernel(swan_mod.SWAN_F16, heads, 16, [old] * B, 191,
                         [L - old for L in Ls]) == PREFILL
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=B, Hq=heads, Hkv=heads, L=Ls, b=16,
                           k_active=[EDGES[i % len(EDGES)] for i in range(B)], dtype="f16",
                           chunks=[old, 191] if old else [191])
    _check(cache, oc, Ls)


@pytest.mark.parametrize("values", ["same", "e4m3"])
@pytest.mark.parametrize("given", [False, True])
def test_prefill_every_fp16_value(gpu_device, swan_mod, torch_mod, values, given):
    """P = identity (values: or given in the rotated basis, P_vo = NULL), k = 128, b = 0: the
    pages hold every finite fp16 value, as it is or as its E4M3 code."""
    torch = torch_mod
    X = _finite_fp16_rows()
    n = X.shape[0]
    assert append_kernel(swan_mod.dtype_code(torch.float16, values), 2, 0, [0] * B, n) == PREFILL
    rows = {0: X, 1: X[::-1].copy()}
    t = [torch.tensor(rows[r], device=gpu_device).expand(B, 2, n, 128).contiguous() for r in (0, 1)]
    eye = torch.eye(128, device=gpu_device).expand(2, 128, 128).contiguous()
    cache = swan_mod.SwanCache(B, 2, 2, 0, n, [128] * B, torch.float16, gpu_device,
                               sparse_values=values)
    cache.append(t[0], t[1], eye, None if given else eye)
    torch.cuda.synchronize()
    for role in (0, 1):
        # the sum with +0 products turns -0 into +0; given rows stay as they are
        want = rows[role] if given and role == 1 else O.to_storage(
            O.rotate(rows[role], np.eye(128)), np.float16)
        want = O.to_e4m3_codes(want) if values == "e4m3" else want
        for bi, h in ((0, 0), (B - 1, 1)):
            idx, val, _, _ = C.unit_pages(cache, bi, h, role, n,
                                          np.uint8 if values == "e4m3" else np.float16)
            assert np.array_equal(idx, np.tile(np.arange(128), (n, 1)))
            assert np.array_equal(val.view(np.uint8), want.view(np.uint8)), (role, bi, h)


@pytest.mark.parametrize("values", ["same", "e4m3"])
@pytest.mark.parametrize("first,b", [(0, 0), (37, 33)])
def test_prefill_values_given(gpu_device, swan_mod, torch_mod, values, first, b):
    """P_vo = NULL and values with their own k, as a layer's prompt has them."""
    torch = torch_mod
    n = 300
    per = [(300, 257, 289, 1)[i % 4] for i in range(B)]
    assert append_kernel(swan_mod.dtype_code(torch.float16, values), 2, b, [first] * B, n,
                         per) == PREFILL
    r = si.rng_for(515, first)
    K = r.standard_normal((B, 2, first + n, 128)).astype(np.float16)
    V = r.standard_normal((B, 2, first + n, 128)).astype(np.float16)
    Pqk = np.stack([si.random_orthogonal(70 + h, 128) for h in range(2)]).astype(np.float32)
    tqk = torch.tensor(Pqk, device=gpu_device)
    ks = [EDGES[i % len(EDGES)] for i in range(B)]
    kv = [EDGES[(3 * i + 5) % len(EDGES)] for i in range(B)]
    cache = swan_mod.SwanCache(B, 2, 2, b, first + n, ks, torch.float16, gpu_device,
                               sparse_values=values, k_value=kv)
    tK, tV = torch.tensor(K, device=gpu_device), torch.tensor(V, device=gpu_device)
    if first:
        cache.append(tK[:, :, :first].contiguous(), tV[:, :, :first].contiguous(), tqk, None)
    cache.append(tK[:, :, first:].contiguous(), tV[:, :, first:].contiguous(), tqk, None,
                 n_new_per_seq=per)
    for bi in range(B):
        L = first + per[bi]
        for h in range(2):
            oc = O.compress_block(K[bi, h, :L], V[bi, h, :L], Pqk[h], np.eye(128), b, ks[bi],
                                  np.float16, values="e4m3" if values == "e4m3" else "t",
                                  k_value=kv[bi])
            C.compare_unit(cache, oc, bi, h, L, np.float16, values=values)


@pytest.mark.parametrize("first,n,per_wave", [(37, 512, 2), (37, 800, 3), (64, 2100, 8)])
def test_prefill_several_units_per_wave(gpu_device, swan_mod, torch_mod, first, n, per_wave):
    """Batches so large that a wave takes several units, onto a cache with tokens."""
    torch = torch_mod
    Bm, H, b = 16, 32, 16
    units = sum((first + n - 1) // 32 - first // 32 + 1 for _ in range(Bm)) * 2 * H
    assert units // (256 * 8 * 4) == per_wave  # what the launch computes
    assert append_kernel(swan_mod.SWAN_F16, H, b, [first] * Bm, n) == PREFILL
    gen = torch.Generator(device=gpu_device).manual_seed(n)
    x = [torch.randn((Bm, H, first + n, 128), device=gpu_device, generator=gen).half()
         for _ in range(2)]
    P = [np.stack([si.random_orthogonal(900 + 50 * r + h, 128) for h in range(H)]).astype(np.float32)
         for r in range(2)]
    tP = [torch.tensor(p, device=gpu_device) for p in P]
    ks = [EDGES[(5 * i) % len(EDGES)] for i in range(Bm)]
    cache = swan_mod.SwanCache(Bm, H, H, b, first + n, ks, torch.float16, gpu_device)
    for lo, hi in ((0, first), (first, first + n)):
        cache.append(x[0][:, :, lo:hi].contiguous(), x[1][:, :, lo:hi].contiguous(), *tP)
    for bi, h in ((0, 0), (3, 31), (7, 12), (15, 5)):
        K, V = (t[bi, h].cpu().numpy() for t in x)
        oc = O.compress_block(K, V, P[0][h], P[1][h], b, ks[bi], np.float16)
        C.compare_unit(cache, oc, bi, h, first + n, np.float16)


def test_prefill_masks_in_one_half(gpu_device, swan_mod, torch_mod, monkeypatch):
    monkeypatch.setattr(si, "random_orthogonal", lambda seed, d: np.eye(d))  # rows as given
    ks = [EDGES[i % len(EDGES)] for i in range(B)]
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=B, Hq=2, Hkv=2, L=260, b=0,
                           k_active=ks, dtype="f16", kv_hook=_one_half)
    _check(cache, oc, [260] * B)


@pytest.mark.parametrize("dtype,values", [("f16", "same"), ("f32", "same"), ("f16", "e4m3")])
@pytest.mark.parametrize("old,new,b", [
    # no new token pruned: blocks of 16, from nothing, a part of the buffer, a full buffer
    (0, 2, 16), (0, 17, 64), (50, 16, 64), (64, 15, 64), (200, 33, 64), (200, 128, 128),
    # pruned: one block, its edges, several workgroups after an eviction launch
    (0, 63, 0), (64, 64, 0), (1, 64, 0), (100, 70, 16), (130, 100, 64), (37, 400, 16),
])
def test_insert_blocks(gpu_device, swan_mod, torch_mod, dtype, values, old, new, b):
    L = old + new
    ks = [40, 77, 128]
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=3, Hq=1, Hkv=1, L=[L, L - 1, L],
                           b=b, k_active=ks, dtype=dtype, values=values,
                           chunks=[old, new] if old else [new])
    _check(cache, oc, [L, L - 1, L], si.np_dtype(dtype), values)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("hook", [_one_half, _extreme_rows])
def test_insert_kept_counts(gpu_device, swan_mod, torch_mod, monkeypatch, dtype, hook):
    if hook is _one_half:
        monkeypatch.setattr(si, "random_orthogonal", lambda seed, d: np.eye(d))
    n = len(EDGES)
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=n, Hq=1, Hkv=1, L=75, b=3,
                           k_active=EDGES, dtype=dtype, kv_hook=hook)
    _check(cache, oc, [75] * n, si.np_dtype(dtype))


def test_insert_fused_eviction_many_units(gpu_device, swan_mod, torch_mod):
    """256 units and up keep a few blocks in one workgroup, which evicts first."""
    Ls = [100 + 7 * (i % 9) for i in range(B)]
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=B, Hq=2, Hkv=2, L=Ls, b=16,
                           k_active=[EDGES[i % len(EDGES)] for i in range(B)], dtype="f16",
                           chunks=[50, 60, 60])
    _check(cache, oc, Ls)
