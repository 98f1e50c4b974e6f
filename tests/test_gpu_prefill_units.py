"""Compress-append of several tokens at once, bit-exact against the oracle: the prefill
kernel (long appends of a large batch) at the edges of its units of 32 positions, and
the insert kernel (everything else) at the edges of its blocks, for every remainder of
k by 8, masks in one half of the dims, ties and extreme rows."""
import numpy as np
import pytest

import swan_inputs as si
from tests import swan_cases as C
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
