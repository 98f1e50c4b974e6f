"""Compress-append of many tokens at the edges of the prefill kernel's units of 32
positions (bit-exact against the oracle): first units that begin in the middle,
one workgroup and several, every remainder of k by 8, the masks whose kept dims
all lie in one half of a token's dims, and ties at the k-th magnitude."""
import numpy as np
import pytest

import swan_inputs as si
from tests import swan_cases as C
from tests.test_gpu_parity import _build, _extreme_rows

pytestmark = pytest.mark.gpu


def _check(cache, oc, L):
    for h in range(2):
        C.compare_unit(cache, oc[0][h], 0, h, L, np.float16)


@pytest.mark.parametrize("old,new,b", [
    (0, 64, 0), (0, 65, 33), (1, 64, 0), (31, 64, 16), (32, 64, 16), (33, 95, 0), (63, 66, 1),
    (17, 255, 0), (0, 256, 0), (0, 257, 64), (5, 515, 31), (100, 1000, 128),
])
def test_unit_edges(gpu_device, swan_mod, torch_mod, old, new, b):
    L = old + new
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=1, Hq=2, Hkv=2, L=L, b=b,
                           k_active=[40], dtype="f16", chunks=[old, new] if old else [new])
    _check(cache, oc, L)


@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 15, 63, 64, 65, 102, 120, 121, 127, 128])
def test_kept_counts(gpu_device, swan_mod, torch_mod, k):
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=1, Hq=2, Hkv=2, L=130, b=8,
                           k_active=[k], dtype="f16", kv_hook=_extreme_rows)
    _check(cache, oc, 130)


def _one_half(K, V):
    """Values of a few equal magnitudes (ties everywhere), in the low half of the dims,
    the high half, or every 8th dim, depending on the token."""
    for X in (K, V):
        n = X.shape[2]
        for t in range(n):
            row = np.zeros(128)
            d = np.arange(128)
            on = (d < 64, d >= 64, d % 8 == t % 8, d % 2 == 0)[t % 4]
            row[on] = np.where(d[on] % 3 == 0, -0.5, 0.25)
            X[:, :, t] = row.astype(X.dtype)


@pytest.mark.parametrize("k", [5, 32, 64, 90])
def test_masks_in_one_half(gpu_device, swan_mod, torch_mod, monkeypatch, k):
    monkeypatch.setattr(si, "random_orthogonal", lambda seed, d: np.eye(d))  # rows as given
    cache, oc, *_ = _build(swan_mod, torch_mod, gpu_device, B=1, Hq=2, Hkv=2, L=100, b=0,
                           k_active=[k], dtype="f16", kv_hook=_one_half)
    _check(cache, oc, 100)
