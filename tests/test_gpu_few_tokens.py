"""Few new tokens of very many (sequence, kv head, role), bit-exact against the oracle on
sampled units: the kernel with one wave per 8 tokens, for tokens that fit the buffer, that
make others leave it (in the same launch, or after an eviction launch) and that are pruned
on arrival, up to two pages, with different lengths and none for some sequences."""
import numpy as np
import pytest

import swan_inputs as si
from oracle import swan_oracle as O
from tests import swan_cases as C
from tests.test_append_plan_host import FEW, INSERT, PREFILL, append_kernel

pytestmark = pytest.mark.gpu

B, H = 64, 16  # 2048 units
EDGES = [1, 7, 8, 9, 40, 63, 64, 77, 120, 121, 127, 128]


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("dtype,values", [("f16", "same"), ("f32", "same"), ("f16", "e4m3")])
@pytest.mark.parametrize("first,n,b,ragged", [
    (0, 2, 16, False), (0, 8, 16, True),           # fit, nothing leaves
    (20, 5, 16, False), (64, 8, 8, True), (9, 7, 16, True),  # fit, the full or filling buffer leaves
    (0, 3, 0, False), (62, 8, 0, True),            # no buffer; over a page's end
    (20, 8, 3, False), (2, 6, 4, True),            # some leave, some are pruned
    (40, 16, 0, False), (40, 32, 0, True), (30, 16, 5, False),  # several waves per unit
])
def test_few_tokens(gpu_device, swan_mod, torch_mod, dtype, values, first, n, b, ragged, given):
    torch = torch_mod
    np_dt = si.np_dtype(dtype)
    per = [(n, n - 1, n, 1, n, 0)[i % 6] if ragged else n for i in range(B)]
    # enough of them for every case
    heads = 2 * H if ragged else H
    assert append_kernel(swan_mod.dtype_code(C.torch_dtype(dtype), values), heads, b, [first] * B,
                         n, per) == FEW
    gen = torch.Generator(device=gpu_device).manual_seed(100 * n + first)
    x = [torch.randn((B, heads, first + n, 128), device=gpu_device, generator=gen).to(
        C.torch_dtype(dtype)) for _ in range(2)]
    P = [np.stack([si.random_orthogonal(300 + 50 * r + h, 128) for h in range(4)]).astype(
        np.float32) for r in range(2)]
    tP = [torch.tensor(p, device=gpu_device).repeat(heads // 4, 1, 1) for p in P]
    if given:
        tP[1], P[1] = None, np.stack([np.eye(128)] * 4)
    ks = [EDGES[i % len(EDGES)] for i in range(B)]
    kv = [EDGES[(5 * i + 3) % len(EDGES)] for i in range(B)]
    cache = swan_mod.SwanCache(B, heads, heads, b, first + n, ks, C.torch_dtype(dtype), gpu_device,
                               sparse_values=values, k_value=kv)
    if first:
        cache.append(x[0][:, :, :first].contiguous(), x[1][:, :, :first].contiguous(), *tP)
    cache.append(x[0][:, :, first:].contiguous(), x[1][:, :, first:].contiguous(), *tP,
                 n_new_per_seq=per)
    for i in range(24):
        bi, h = (11 * i) % B, (7 * i + i // 4) % heads
        L = first + per[bi]
        if L == 0:
            continue
        K, V = (t[bi, h, :L].cpu().numpy() for t in x)
        oc = O.compress_block(K, V, P[0][h % 4], P[1][h % 4], b, ks[bi], np_dt,
                              values="e4m3" if values == "e4m3" else "t", k_value=kv[bi])
        C.compare_unit(cache, oc, bi, h, L, np_dt, values=values)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("first,b", [(0, 0), (37, 16), (70, 200)])
def test_sequences_of_other_lengths(gpu_device, swan_mod, torch_mod, dtype, first, b):
    """The insert kernel for sequences with different numbers of blocks, and so many of
    some that a workgroup takes several: every sequence's units, also those of none."""
    torch = torch_mod
    heads, np_dt = 16, si.np_dtype(dtype)
    per = [(1, 700, 0, 64, 65, 40, 127, 1, 513, 3)[i % 10] for i in range(B - 4)] + [0, 900, 20, 0]
    assert append_kernel(swan_mod.dtype_code(C.torch_dtype(dtype), "same"), heads, b, [first] * B,
                         900, per) == INSERT
    gen = torch.Generator(device=gpu_device).manual_seed(first)
    x = [torch.randn((B, heads, first + 900, 128), device=gpu_device, generator=gen).to(
        C.torch_dtype(dtype)) for _ in range(2)]
    P = [np.stack([si.random_orthogonal(400 + 50 * r + h, 128) for h in range(heads)]).astype(
        np.float32) for r in range(2)]
    tP = [torch.tensor(p, device=gpu_device) for p in P]
    ks = [EDGES[i % len(EDGES)] for i in range(B)]
    cache = swan_mod.SwanCache(B, heads, heads, b, first + 900, ks, C.torch_dtype(dtype), gpu_device)
    if first:
        cache.append(x[0][:, :, :first].contiguous(), x[1][:, :, :first].contiguous(), *tP)
    cache.append(x[0][:, :, first:].contiguous(), x[1][:, :, first:].contiguous(), *tP,
                 n_new_per_seq=per)
    for bi in list(range(12)) + list(range(B - 5, B)):
        L, h = first + per[bi], (3 * bi) % heads
        if L == 0:
            continue
        K, V = (t[bi, h, :L].cpu().numpy() for t in x)
        oc = O.compress_block(K, V, P[0][h], P[1][h], b, ks[bi], np_dt)
        C.compare_unit(cache, oc, bi, h, L, np_dt)


def _not_numbers(torch, x):
    rows = x.view(torch.int16)
    for i, v in enumerate((0x7E00, 0xFE00, 0x7D01, 0x7FFF, 0x7C00, 0xFC00, 0xFD03)):
        v -= 65536 if v > 32767 else 0
        rows[0, 0, i, 5 * i + 1] = v
        rows[1, -2, i] = v
        rows[1, -1, i + 8, 3] = v


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("buffer", [0, 5, 64])
def test_not_numbers(gpu_device, swan_mod, torch_mod, buffer, given):
    """Rows with infinities and NaNs of any bits: the bytes of an append of all tokens are
    those of one token after another; RoPE gives one NaN, with either sign."""
    torch = torch_mod
    gen = torch.Generator(device=gpu_device).manual_seed(3)
    x = torch.randn((2, 4, 24, 128), device=gpu_device, generator=gen).half()
    _not_numbers(torch, x)
    P = torch.tensor(np.stack([si.random_orthogonal(70 + h, 128) for h in range(4)]),
                     dtype=torch.float32, device=gpu_device)
    caches = [swan_mod.SwanCache(2, 4, 4, buffer, 64, [40, 128], torch.float16, gpu_device)
              for _ in range(2)]
    assert append_kernel(swan_mod.SWAN_F16, 4, buffer, [0, 0], 24) == INSERT
    caches[0].append(x, x, P, None if given else P)
    for t in range(24):
        one = x[:, :, t:t + 1].contiguous()
        caches[1].append(one, one, P, None if given else P)
    for a, b in zip(*([c.k_pages, c.v_pages, c.k_ring.view(torch.int16), c.v_ring.view(torch.int16)]
                      for c in caches)):
        assert torch.equal(a, b)
    y = swan_mod.rope(x, [3, 1000], 10000.0)
    nan = y.view(torch.int16)[y.isnan()] & 0x7FFF
    assert nan.numel() and bool((nan == 0x7E00).all())


@pytest.mark.parametrize("buffer", [0, 40])
def test_not_numbers_of_a_prompt(gpu_device, swan_mod, torch_mod, buffer):
    """The prefill kernel's bytes of such rows are the insert kernel's, sequence by sequence."""
    torch = torch_mod
    gen = torch.Generator(device=gpu_device).manual_seed(4)
    x = torch.randn((B, 2, 300, 128), device=gpu_device, generator=gen).half()
    _not_numbers(torch, x)
    P = torch.tensor(np.stack([si.random_orthogonal(70 + h, 128) for h in range(2)]),
                     dtype=torch.float32, device=gpu_device)
    new = lambda n: swan_mod.SwanCache(n, 2, 2, buffer, 300, [40] * n, torch.float16, gpu_device)
    assert append_kernel(swan_mod.SWAN_F16, 2, buffer, [0] * B, 300) == PREFILL
    all_, one = new(B), new(1)
    all_.append(x, x, P, P)
    for i in (0, 1, 2):
        one.seq_len = [0]
        one.append(x[i:i + 1], x[i:i + 1], P, P)
        for a, b in ((all_.k_pages, one.k_pages), (all_.v_pages, one.v_pages),
                     (all_.k_ring.view(torch.int16), one.k_ring.view(torch.int16)),
                     (all_.v_ring.view(torch.int16), one.v_ring.view(torch.int16))):
            assert torch.equal(a.reshape(B, -1)[i], b.flatten()), i


def test_time_of_uneven_groups(gpu_device, swan_mod, torch_mod):
    """8 blocks of every unit and one block more, in two groups of workgroups: the time of
    the blocks, whatever processors their groups fall to (512 of 1024 tokens took 0.91 of
    the time when the long groups shared half of them)."""
    torch = torch_mod
    heads, first, us = 32, 1000, {}
    P = torch.eye(128, device=gpu_device).expand(heads, 128, 128).contiguous()
    for n in (512, 1024):
        cache = swan_mod.SwanCache(B, heads, heads, 0, first + n, [48] * B, torch.float32, gpu_device)
        x = torch.randn((B, heads, n, 128), device=gpu_device)
        for _ in range(4):
            cache.seq_len = [first] * B
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            cache.append(x, x, P, P)
            e[1].record()
            torch.cuda.synchronize()
            us[n] = min(us.get(n, 1e9), e[0].elapsed_time(e[1]))
    assert us[512] <= 0.7 * us[1024], us
